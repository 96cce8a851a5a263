"""The order of the items of attn_short.hpp and attn_sparse.hpp (set_items, item_of): every block of every head once, and, with lists, what an XCD
works on at a time shares few KV heads, whatever their number.  CPU only: the header's host code, compiled here."""
import os
import subprocess

import numpy as np
import pytest

from paper_2604_12798_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")

MAIN = """
#include "common.hpp"
#include <cstdio>
int main(int, char** v) {
    Params p{};
    p.B = atoi(v[1]); p.Hq = atoi(v[2]); p.Hkv = atoi(v[3]); p.Tr = atoi(v[4]);
    set_items(p, atoi(v[5]) != 0);
    for (int id = 0; id < p.B * p.Hq * p.Tr; ++id) {
        const Item it = item_of(p, id);
        printf("%d %d %d\\n", it.head, it.kv, it.i);
    }
}
"""


@pytest.fixture(scope="module")
def items(tmp_path_factory):
    d = tmp_path_factory.mktemp("items")
    (d / "main.hip").write_text(MAIN)
    subprocess.run([HIPCC] + [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")] + ["-I" + build.CSRC, "--offload-host-only", "-o", str(d / "a"),
                   str(d / "main.hip")], check=True, capture_output=True)

    def run(*args):
        out = subprocess.run([str(d / "a"), *map(str, args)], check=True, capture_output=True, text=True).stdout
        return np.array(out.split(), dtype=np.int64).reshape(-1, 3)
    return run


# KV heads: fewer than eight, eights, one more and less, many
@pytest.mark.parametrize("B,Hq,Hkv,Tr", [(1, 4, 1, 5), (1, 7, 7, 9), (2, 32, 4, 3), (1, 9, 9, 40), (1, 45, 15, 17), (3, 22, 11, 1), (1, 134, 67, 42), (7, 19, 19, 34), (5, 96, 32, 13)])
@pytest.mark.parametrize("lists", [0, 1])
def test_items(items, B, Hq, Hkv, Tr, lists):
    got, g, G = items(B, Hq, Hkv, Tr, lists), Hq // Hkv, B * Hkv
    head, kv, i = got.T
    assert (kv == head // g).all() and i.min() >= 0 and i.max() == Tr - 1
    assert len(np.unique(head * Tr + i)) == len(got) == B * Hq * Tr
    # a head's late blocks first
    for h in (0, G * g // 2, G * g - 1):
        assert (np.diff(i[head == h]) == -1).all()
    if not lists or G < 8:
        return
    # 64 items of an XCD at a time (two workgroups to a unit): of the lists', those of the KV heads that they are enough for, and one that
    # they end in; the rest, at the front, are of fewer than eight KV heads
    rest = (G & 7) * g * Tr
    assert len(np.unique(kv[:rest])) == (G & 7)
    for x in range(8):
        own = kv[rest:][np.arange(rest, len(got)) % 8 == x]
        for a in range(0, len(own), 64):
            assert len(np.unique(own[a:a + 64])) <= -(-64 // (g * Tr)) + 1
