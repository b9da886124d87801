"""CPU check of the home slots of the small group-bys' LDS tables
(csrc/gq_slot_hash.h): structured keys must not crowd a few slots.  A small C++
driver that includes the header is compiled with g++; it fills a table as the
kernels do: by groups of four slots, at most 16 groups from the home group, or
slot by slot, at most 64 from the home slot (the batched form)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_09226_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "gq_slot_hash.h"
int main(int argc, char **argv) {
    const int SIZE = argc > 1 ? std::atoi(argv[1]) : 4;          // slots read together
    const int GROUPS = 1024 / SIZE, REACH = 64 / SIZE;
    int n;
    while (std::scanf("%d", &n) == 1) {
        std::vector<int> fill(GROUPS, 0);
        long long reads = 0;
        int lost = 0;
        for (int i = 0; i < n; ++i) {
            long long a, b;
            if (std::scanf("%lld %lld", &a, &b) != 2) return 1;
            const unsigned x = gq_slot_hash(static_cast<uint64_t>(a), static_cast<uint32_t>(b));
            int g = static_cast<int>(x >> 22) / SIZE, p = 0;
            while (p < REACH && fill[g] == SIZE) { g = (g + 1) % GROUPS; ++p; }
            if (p == REACH) ++lost;
            else ++fill[g];
            reads += p + 1;
        }
        std::printf("%lld %d\n", reads, lost);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)])
    return str(exe)


def u32(v):
    return v % (1 << 32)


R = range(512)
STRIDES = list(range(1, 64)) + [100, 987, 1000, 1597, 2584, 3600, 4181, 10_000, 10_946, 28_657, 86_400, 1_000_000] + \
    [1 << s for s in range(6, 23)]
KEYS = {
    "20 x 25": [(a, b) for a in range(20) for b in range(25)],
    "22 x 23": [(a, b) for a in range(22) for b in range(23)],
    "100 (i, -i)": [(i, -i) for i in range(100)],
    "512 (i, 511 - i)": [(i, 511 - i) for i in R],
    "(i, i)": [(i, i) for i in R],
    "(i, -3 i)": [(i, -3 * i) for i in R],
    "(i << 32, -i)": [(i << 32, -i) for i in R],
    "(1000 i, 1000 (511 - i))": [(1000 * i, 1000 * (511 - i)) for i in R],
    **{f"key64 {s} i": [(s * i, 0) for i in R] for s in STRIDES},
    **{f"key32 -{s} i": [(u32(-s * i), 0) for i in R] for s in STRIDES},      # (a 32-bit key is the low word)
    **{f"(i // 16, {s} (i % 16))": [(i // 16, s * (i % 16)) for i in R] for s in STRIDES},
}
RUNS = {f"{a}..": [(a + i, 0) for i in R] for a in (0, 1, 200, 1000, 65_300, 1_234_567, 123_456_789_012)} | \
    {f"key32 {a}..": [(u32(a + i), 0) for i in R] for a in (-511, -300, (1 << 31) - 256)}


# At most half of the 1024 slots are taken, so a group of four overflows for
# few keys whatever their order (Poisson of mean 2: about 1.05 reads a key for
# random home slots); twice that is a crowd.
# (Runs of consecutive codes: runs of 256 put at most two keys in a group, so
# hardly any of 512 codes, whole or cut by the runs' edges, miss theirs.)
@pytest.mark.parametrize("sets,most", [(KEYS, 2.1), (RUNS, 1.05)])
def test_structured_keys_spread(driver, sets, most):
    text = "".join(f"{len(k)}\n" + "".join(f"{a} {b}\n" for a, b in k) for k in sets.values())
    out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert len(out) == 2 * len(sets)
    bad = {}
    for (name, keys), reads, lost in zip(sets.items(), out[0::2], out[1::2]):
        assert len(set(keys)) == len(keys)
        if int(lost) or int(reads) > most * len(keys):
            bad[name] = (int(reads) / len(keys), int(lost))
    assert not bad, bad


# Slot by slot, random home slots of 512 keys in 1024 slots take 1.5 reads a key.
def test_structured_codes_spread_over_single_slots(driver):
    sets = {k: v for k, v in (KEYS | RUNS).items() if all(b == 0 and a < 1 << 32 for a, b in v)}
    assert len(sets) > 50
    text = "".join(f"{len(k)}\n" + "".join(f"{a} {b}\n" for a, b in k) for k in sets.values())
    out = subprocess.run([driver, "1"], input=text, capture_output=True, text=True, check=True).stdout.split()
    bad = {}
    for (name, keys), reads, lost in zip(sets.items(), out[0::2], out[1::2]):
        if int(lost) or int(reads) > 3.0 * len(keys):
            bad[name] = (int(reads) / len(keys), int(lost))
    assert not bad, bad
