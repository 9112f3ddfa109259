"""The least share of the attention kernel's even split (kernels.h), on the host.

The kernel compares a head's tile count with limits the host has worked out; here the rule is restated per
case, from the averages it is about, and both agree over the range of batches.
"""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
int main() {
  int total, seqs, hkv, dim, rows;
  while (std::scanf("%d %d %d %d %d", &total, &seqs, &hkv, &dim, &rows) == 5)
    std::printf("%d\n", spexis::attn_least_tiles(spexis::attn_least(seqs, hkv, dim, rows), total));
}
"""


@pytest.fixture(scope="module")
def least(tmp_path_factory):
    d = tmp_path_factory.mktemp("shares")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2609_34370_amd", "csrc"), str(d / "p.cpp"), "-o", str(d / "p")],
                   check=True)

    def run(cases):
        text = "\n".join(" ".join(map(str, c)) for c in cases)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]

    return run


def restated(total, seqs, hkv, dim, rows):
    nt, everywhere = total / seqs, total * hkv
    if nt >= 1024 or (seqs == 1 and everywhere >= 2048 and nt >= 3):
        return 6
    if everywhere >= 4096 and dim == 128 and rows <= 32 and nt >= 8:
        return 6
    if nt >= (256 if rows > 32 else 512) or (everywhere >= 2048 and nt >= 3):
        return 4
    return 4 if (rows > 32 or (rows >= 8 and everywhere >= 1024)) and 3 <= nt < 5 else 2


def test_least_share_is_the_stated_rule(least):
    rng = random.Random(1)
    cases = []
    for _ in range(4000):
        seqs = int(2 ** rng.uniform(0, 10))
        total = max(1, int(seqs * 2 ** rng.uniform(0, 12)))
        cases.append((total, seqs, rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 32]), rng.choice([64, 128]),
                      rng.randint(1, 64)))
    for seqs in (1, 2, 64, 512):   # the limits themselves, and one tile to either side
        for nt in (2, 3, 4, 5, 8, 256, 512, 1024):
            cases += [(max(1, seqs * nt + e), seqs, hkv, dim, r) for e in (-1, 0, 1) for hkv in (1, 8) for dim in (64, 128)
                      for r in (4, 8, 32, 33)]
    assert least(cases) == [restated(*c) for c in cases]


@pytest.mark.parametrize("total,seqs,hkv", [
    (512, 64, 1),     # 64 sequences of 256 keys, one KV head
    (256, 128, 1),    # 128 of 64 keys
    (512, 16, 1),     # 16 of 1024 keys
    (512, 256, 2),
])
def test_short_sequences_keep_shares_of_two_tiles(least, total, seqs, hkv):
    # longer shares left waves idle and took 1.14 to 1.48 times as long
    assert least([(total, seqs, hkv, 128, 20)]) == [2]


def test_batches_past_the_integer_range(least):
    # limits of hundreds of tiles a sequence saturate
    assert least([(2 ** 31 - 1, 2 ** 28, 1, 128, 20), (2 ** 30, 2 ** 30, 1, 64, 63)]) == [6, 2]
