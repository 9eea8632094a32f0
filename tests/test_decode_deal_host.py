"""How a split decode deals its key ranges to requests of uneven lengths (pic_bounds.h), on the CPU: the
candidate sizes run from the mean to the longest request in n_splits ranges, which always fits; the
size taken is the first that fits the launch, and its ranges cover every request and have workgroups
and partial slots of their own.  (The kernels' own arithmetic is compared on the GPU.)"""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
SRC = r"""
#include <cstdio>
#include "pic_bounds.h"
int main() {
  int total, longest, n_splits, batch;
  while (std::scanf("%d %d %d %d", &total, &longest, &n_splits, &batch) == 4) {
    const pic::RangeCandidates rc = pic::decode_range_candidates(total, longest, n_splits, batch);
    for (int i = 0; i < pic::kDecodeDealt; ++i) std::printf("%d ", rc.at(i));
    std::printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def candidates(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ in this image")
    d = tmp_path_factory.mktemp("deal")
    (d / "deal.cpp").write_text(SRC)
    subprocess.run([CLANG, "-std=c++17", "-O1", f"-I{ROOT}/include", f"-I{ROOT}/paper_2607_28069_amd/csrc",
                    str(d / "deal.cpp"), "-o", str(d / "deal")], check=True, timeout=120)

    def run(rows):
        r = subprocess.run([str(d / "deal")], input="\n".join(" ".join(map(str, x)) for x in rows), text=True,
                           capture_output=True, check=True, timeout=60)
        return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]

    return run


def test_ranges_fit_and_cover(candidates):
    rng = random.Random(0)
    cases = []
    for _ in range(2000):
        batch, n_splits = rng.randint(2, 64), rng.choice([8, 9, 16, 31, 32, 64, 1000])
        top = rng.choice([1, 3, 64, 300, 5000, 1 << 24])
        cases.append((n_splits, [rng.randint(1, top) for _ in range(batch)]))
    cases += [(8, [1] * 64), (8, [1 << 24] * 64), (16, [1] * 63 + [1 << 24]), (8, [8, 1])]
    got = candidates([(sum(u), max(u), s, len(u)) for s, u in cases])
    assert len(got) == len(cases)
    for (s, u), cs in zip(cases, got):
        ranges = lambda c: sum(-(-x // c) for x in u)
        budget = s * len(u)
        assert cs == sorted(cs) and cs[0] >= 1
        assert cs[-1] == -(-max(u) // min(s, max(u))) and ranges(cs[-1]) <= budget
        assert cs[0] * min(s, max(u)) * len(u) >= sum(u)   # (nothing smaller than the mean could fit)


def test_size_taken_ranges_and_places(candidates):
    rng = random.Random(1)
    cases = []
    for _ in range(200):
        batch, n_splits = rng.randint(2, 64), rng.choice([8, 9, 16, 31])
        top = rng.choice([64, 75, 300, 5000])
        cases.append((n_splits, rng.choice([1, 3]), [rng.randint(1, top) for _ in range(batch - 1)] + [top]))
    for (s, hq, u), cs in zip(cases, candidates([(sum(u), max(u), s, len(u)) for s, _, u in cases])):
        fits = [sum(-(-x // c) for x in u) <= s * len(u) for c in cs]
        size = cs[fits.index(True)]
        assert all(not f for f in fits[:fits.index(True)]) and all(fits[fits.index(True):])   # (larger ones fit too)
        n = [-(-x // size) for x in u]
        first = [sum(n[:b]) for b in range(len(u))]
        workgroups, slots = set(), set()
        for b, x in enumerate(u):
            assert n[b] >= 1 and (n[b] - 1) * size < x <= n[b] * size        # every range holds keys, together all
            for h in range(hq):
                for r in range(n[b]):
                    workgroups.add(first[b] * hq + h * n[b] + r)             # [request][head][range], hq kv heads
                    slots.add(first[b] * hq + h * n[b] + r)
        assert len(slots) == len(workgroups) == sum(n) * hq
        assert max(slots) < s * len(u) * hq
