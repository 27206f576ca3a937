"""The tiled GEMMs' choice of tile shape and split plan (csrc/gemm_plan.h), asked
on the host: what the sizes of the GPU tests take, and what has to hold for every
size."""
import random
import shutil
import subprocess

import pytest
from tile_sizes import EIGHT, ERR_EIGHT, ERR_FOUR, FOUR, GELU_EIGHT, GELU_FOUR

from paper_2609_39056_amd import _build

SRC = """
#include "gemm_plan.h"
#include <stdio.h>
using namespace sq;
int main() {
  int bits, pc, M, K, N, cus;
  double share;  // of the queried workspace that the call has
  while (scanf("%d %d %d %d %d %d %lf", &bits, &pc, &M, &K, &N, &cus, &share) == 7) {
    const size_t query = pipe_partial_bytes(M, N, K, cus), have = static_cast<size_t>(query * share);
    const Choice c = bits == 4 ? choose8(M, N, K, cus, have)
                     : pc      ? choose16<true>(M, N, K, cus, have)
                               : choose16<false>(M, N, K, cus, have);
    static const int rows[] = {256, 128, 64, 64}, cols[] = {128, 128, 128, 64};
    printf("%d %d %d %d %d %zu %zu\\n", rows[c.tile], cols[c.tile], c.plan.ntiles, c.plan.ndp, c.plan.split, have,
           err_parts(c));
  }
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("choice")
    (d / "choice.cpp").write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{_build.CSRC}", str(d / "choice.cpp"), "-o", str(d / "choice")], check=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows) + "\n"
        out = subprocess.run([str(d / "choice")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return ask


def name(c):
    bm, bn, ntiles, ndp, split = c[:5]
    return f"{bm}x{bn} " + ("whole" if split == 1 else "split" if ndp == 0 else "tail")


@pytest.mark.parametrize("sizes", [EIGHT, GELU_EIGHT, ERR_EIGHT], ids=["linear", "gelu", "error"])
def test_choice_of_the_tested_sizes_8bit(choose, sizes):
    got = choose([(8, pc, *s, 256, 1.0) for s in sizes for pc in (0, 1)])
    assert {s: (name(got[2 * i]), name(got[2 * i + 1])) for i, s in enumerate(sizes)} == sizes


@pytest.mark.parametrize("sizes", [FOUR, GELU_FOUR, ERR_FOUR], ids=["linear", "gelu", "error"])
def test_choice_of_the_tested_sizes_4bit(choose, sizes):
    got = choose([(4, 0, *s, 256, 1.0) for s in sizes])
    assert {s: name(c) for s, c in zip(sizes, got)} == sizes


def test_every_kernel_is_tested(choose):
    """Shapes x (whole, split, tail) that the rules can reach at all."""
    kinds = {"whole", "split", "tail"}
    every = {f"{t} {k}" for t in ("128x128", "64x128", "64x64") for k in kinds} | {"256x128 whole", "256x128 tail"}
    for sizes in (EIGHT, ERR_EIGHT):
        assert {v[0] for v in sizes.values()} == every
        assert {v[1] for v in sizes.values()} == every - {"64x128 tail"}
    four = {f"{t} {k}" for t in ("128x128", "64x128", "64x64") for k in ("whole", "split")} | {"128x128 tail"}
    assert set(FOUR.values()) == set(GELU_FOUR.values()) == set(ERR_FOUR.values()) == four


def test_small_tiles_have_to_promise_more(choose):
    """Measured slower on the smaller tiles than on 128 x 128 (per channel, us):
    short contractions over more than a round of tiles, and long ones on 64 x 64
    or split tiles."""
    slow = [(2227, 384, 8576), (1855, 256, 10624), (3619, 256, 5440), (7866, 512, 4608),  # 0.91-0.96 of 128 x 128
            (4142, 12160, 960), (4716, 7168, 832), (5474, 6016, 704), (293, 13568, 4032)]  # 0.90-0.95
    fast = [(4567, 384, 1920), (1796, 512, 8896), (1536, 8192, 2048), (756, 6784, 1280)]  # 1.04-1.2
    got = [name(c).split()[0] for c in choose([(8, 1, *s, 256, 1.0) for s in slow + fast])]
    assert got[:len(slow)] == ["128x128"] * len(slow)
    assert "128x128" not in got[len(slow):]


def test_plans_are_well_formed(choose):
    """Every output in one tile, ranges of at least two stages, partial sums within
    the workspace at hand, the error epilogue's sums within the fp32 output's
    place, and one plan for every workspace of the queried size or more."""
    r = random.Random(5)
    rows = []
    for _ in range(4000):
        M, K, N = int(2 ** r.uniform(7.1, 15)), 128 * int(2 ** r.uniform(0, 7)), 64 * int(2 ** r.uniform(0, 8.5))
        bits, pc = r.choice([(8, 0), (8, 1), (4, 0)])
        rows.append((bits, pc, M, K, N, r.choice([256, 256, 104, 32]), r.choice([0.0, 0.3, 1.0])))
    rows += [(b, p, 1 << 24, 128, 1 << 20, 256, 1.0) for b, p in ((8, 0), (8, 1), (4, 0))]
    for (bits, pc, M, K, N, cus, share), (bm, bn, ntiles, ndp, split, have, parts) in zip(rows, choose(rows)):
        assert ntiles == -(-M // bm) * -(-N // bn) < 2**31
        assert 0 <= ndp <= ntiles and (split == 1) == (ndp == ntiles)
        if split > 1:
            assert K // 128 // split >= 2
            assert (ntiles - ndp) * split * bm * bn * 4 <= have
        assert parts * 8 <= M * N * 4
    eight = [row for row in rows if row[0] == 8]
    assert choose([row[:6] + (1.0,) for row in eight]) == [
        c[:5] + (w[5],) + c[6:] for c, w in zip(choose([row[:6] + (3.0,) for row in eight]), choose([row[:6] + (1.0,) for row in eight]))]
