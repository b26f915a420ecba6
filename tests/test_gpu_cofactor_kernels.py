"""The kernels with the uniform-cofactor test, at sizes where the library runs
them: counts and lists from 2^18 tiles on, with the test in the wave or (fewer
than one tile in 128 expected to live) in a launch of its own, vectors from
2^13 tiles and 13 clauses for each word per lane (with a general part 2^16 and 24) on.  Against the oracle where it
is quick, else against the same program without the test."""

import itertools
import random

import numpy as np
import pytest

import oracle
from formula_gen import random_cnf
from test_gpu_enumerate import lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1310_6978_amd import fbg
    return fbg


def tile_clauses(rng, lo, n, count, width):
    """count distinct clauses over x_lo .. x_(n-1), all true under one assignment."""
    plant = {v: rng.random() < 0.5 for v in range(lo, n)}
    out = set()
    while len(out) < count:
        vs = sorted(rng.sample(range(lo, n), width))
        keep = rng.choice(vs)
        out.add(" | ".join(("x%d" if (plant[v] if v == keep else rng.random() < 0.5) else "~x%d") % v for v in vs))
    return "".join(c + "\n" for c in sorted(out))


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("wpl", [1, 2, 4, 8, 16, 32])
def test_counts_and_lists(F, wpl, sparse, general):
    rng = random.Random(wpl)
    log2w = wpl.bit_length() - 1
    n, lo = 29 + log2w, 11 + log2w          # 2^18 tiles
    text = tile_clauses(rng, lo, n, 50 if sparse else 9, 3)          # one tile in 800, in 3
    text += random_cnf(rng, n, 2 * n, (3, 4)) + "x0\n~x3 | x1\nx5 | ~x7\n"
    if general:
        text += "(x1 ^ x9 ^ x%d) | (x4 & ~x13)\n" % (n - 1)
    p, q = F.Program(text, n), F.Program(text, n)
    p.set_tuning(wpl, cofactor=True)
    q.set_tuning(wpl)
    assert F.program_tiles(p, wpl) == 1 << 18
    total = int(F.count(q).item())
    if n == 29:
        assert total == oracle.count(text, n)
    assert total > 0
    print("cofactor", wpl, sparse, general, total, flush=True)
    assert int(F.count(p).item()) == total
    want = F.enumerate_models(q, total + 1)[0].cpu().numpy()[:total].view(np.uint64)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, [total + 1, 10])


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("wpl", [1, 2, 4, 8, 16, 32])
def test_vectors(F, wpl, general):
    rng = random.Random(wpl + 100)
    log2w = wpl.bit_length() - 1
    tiles = 1 << 16 if general and wpl < 32 else 1 << 13
    lo = 11 + log2w
    n = lo + tiles.bit_length() - 1
    need = (24 if general else 13) * wpl
    m = need + wpl                          # (a few of them may be implied and go)
    text = tile_clauses(rng, lo, n, 7, 3) + random_cnf(rng, n, m, (3 + log2w, 4 + log2w))
    if general:
        text += "(x1 ^ x9 ^ x%d) | (x4 & ~x13)\n" % (n - 1)
    p = F.Program(text, n)
    assert p.info["n_clause_instr"] >= need and F.program_tiles(p, wpl) == tiles
    got = F.eval_dnf(p, words_per_lane=wpl, cofactor=True).cpu().numpy().view(np.uint64)
    want = oracle.dnf(text, n) if n <= 26 else F.eval_dnf(p, words_per_lane=wpl).cpu().numpy().view(np.uint64)
    assert want.any() and np.array_equal(got, want)


@pytest.mark.parametrize("sparse", [False, True])
def test_more_than_2_32_tiles(F, sparse):
    """2^33 tiles (44 letters at one word per lane), nearly all of their bits fixed by
    unit clauses or by pairs of clauses with a lane literal, which the test does not
    see."""
    import torch
    n = 44
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("the temporaries take 96 GiB")
    free = [11, 14, 43]
    fixed = [k for k in range(11, n) if k not in free]
    text = "".join("x%d\n" % k if sparse or i < 6 else "x%d | x5\nx%d | ~x5\n" % (k, k) for i, k in enumerate(fixed))
    text += "".join("x%d\n" % k for k in range(3, 11)) + "x0 | x2\n"
    p = F.Program(text, n)
    p.set_tuning(1, cofactor=True)
    base = sum(1 << k for k in list(range(3, 11)) + fixed)
    want = np.array(sorted(base | x | sum(b << k for b, k in zip(top, free)) for x in range(8) if x & 5
                           for top in itertools.product((0, 1), repeat=3)), dtype=np.uint64)
    print("2^33 tiles", sparse, len(want), flush=True)
    assert int(F.count(p).item()) == len(want)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, [len(want) + 1])
