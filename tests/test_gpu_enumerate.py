"""Enumeration at the edges of its paths: lists staged through LDS in one and
in many flushes, tiles cut into units, blocks that find their own positions
up to 4096 units (16384 tiles of a stored vector) and the list of the units
with models beyond, programs of a batch that start inside a block of that
list, truncated lists.  Against the oracle."""

import random

import numpy as np
import pytest

import oracle
import workloads
from formula_gen import many_registers, random_cnf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1310_6978_amd import fbg
    return fbg


def lists(call, want, caps):
    """call(capacity, out, total) fills out; the first `capacity` models and
    no word beyond them are written."""
    import torch
    for cap in caps:
        out = torch.full((cap + 3,), -7, dtype=torch.int64, device="cuda")
        tot = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        call(cap, out, tot)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        k = min(cap, len(want))
        assert int(tot.item()) == len(want)
        assert np.array_equal(got[:k].view(np.uint64), want[:k])
        assert (got[k:] == -7).all()


def formulas():
    rng = random.Random(11)
    return {
        "half": lambda n: "x%d\n" % (n - 1),                  # every word of half of the tiles full
        "odd": lambda n: " ^ ".join("x%d" % k for k in range(n)) + "\n",   # 16 models in every word
        "sparse": lambda n: random_cnf(rng, n, 3 * n, (2, 4)),
        "one": lambda n: "\n".join("%sx%d" % ("~" if k % 3 == 0 else "", k) for k in range(n)) + "\n",
        "general": lambda n: many_registers(rng, n, 9),
    }


@pytest.mark.parametrize("kind", ["half", "odd", "sparse", "one", "general"])
@pytest.mark.parametrize("wpl", [1, 2, 8, 16, 32])
@pytest.mark.parametrize("n", [3, 11, 13, 17])
def test_lists(F, kind, wpl, n):
    text = formulas()[kind](max(n, 4) if kind == "general" else n)
    n = max(n, 4) if kind == "general" else n
    p = F.Program(text, n)
    p.set_tuning(wpl)
    want, c = oracle.models(text, n)
    dnf = F.eval_dnf(p)
    caps = [c + 1, max(0, c // 2), 0]
    print("lists", kind, wpl, n, c, flush=True)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, caps)
    lists(lambda cap, out, tot: F.enumerate_dnf(dnf, n, cap, out=out, total=tot), want, caps)


@pytest.mark.parametrize("n,wpl", [(22, 1), (23, 1), (24, 1), (23, 8), (25, 16), (28, 32), (29, 1)])
@pytest.mark.parametrize("cofactor", [False, True])
def test_tile_thresholds(F, n, wpl, cofactor):
    """4096 units (n = 23 at one word per lane) are the last without a list;
    tiles are cut into units of four rows and more below 32768 units; from
    2^18 tiles (n = 29) the cofactor test has a launch of its own."""
    text = workloads.random_3cnf(n, 3 * n, n)[0]
    p = F.Program(text, n)
    p.set_tuning(wpl, cofactor=cofactor)
    ref = F.Program(text, n)
    want = F.eval_dnf(ref)
    want = np.flatnonzero(np.unpackbits(want.cpu().numpy().view(np.uint8), bitorder="little")).astype(np.uint64)
    assert len(want) == oracle.count(text, n)
    print("thresholds", n, wpl, cofactor, len(want), flush=True)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, [len(want) + 1, 100])


@pytest.mark.parametrize("n", [27, 28, 30, 31])
def test_stored_vector_thresholds(F, n):
    """16384 tiles (n = 27 at 1 KiB, n = 30 at 8 KiB) are the last without a
    list.  Models spread out, and crowded into the last tiles."""
    for text in (workloads.random_3cnf(n, 3 * n, n)[0], "\n".join("x%d" % k for k in range(17, n)) + "\nx0 ^ x5\n"):
        p = F.Program(text, n)
        dnf = F.eval_dnf(p)
        total = int(F.count(p).item())
        want = F.enumerate_models(p, total + 1)[0].cpu().numpy()[:total].view(np.uint64)
        assert total > 0 and (np.diff(want.astype(np.int64)) > 0).all()
        print("stored", n, total, flush=True)
        lists(lambda cap, out, tot: F.enumerate_dnf(dnf, n, cap, out=out, total=tot), want, [total + 1, 10])


def test_more_blocks_than_are_summed(F):
    """Over 1024 blocks of the list (n = 33 at one word per lane: 2048)."""
    text = workloads.random_3cnf(33, 132, 5)[0]
    p, q = F.Program(text, 33), F.Program(text, 33)
    q.set_tuning(32)
    p.set_tuning(1)
    total = int(F.count(q).item())
    a, ta = F.enumerate_models(p, total + 1)
    b, tb = F.enumerate_models(q, total + 1)
    assert total > 0 and int(ta.item()) == int(tb.item()) == total
    assert np.array_equal(a.cpu().numpy()[:total], b.cpu().numpy()[:total])


@pytest.mark.parametrize("wpl", [0, 1])
def test_batch_programs_inside_list_blocks(F, wpl):
    import torch
    rng = random.Random(3)
    ns = [5, 13, 20, 11, 22, 17, 12, 21]
    texts = [random_cnf(rng, n, 2 * n, (2, 4)) if i % 3 else "x%d ^ x0\n" % (n - 1) for i, n in enumerate(ns)]
    progs = [F.Program(t, n) for t, n in zip(texts, ns)]
    wants = [oracle.models(t, n)[0] for t, n in zip(texts, ns)]
    b = F.Batch(progs, words_per_lane=wpl)
    b.set_dnf_outputs([torch.empty(F.dnf_words(n), dtype=torch.int64, device="cuda") for n in ns])
    outs = [torch.full((len(w) + 2,), -7, dtype=torch.int64, device="cuda") for w in wants]
    b.set_enum_outputs(outs)
    for _ in range(2):
        counts = b.eval_dnf()
        b.enumerate()
        torch.cuda.synchronize()
        for o, w, c in zip(outs, wants, counts.cpu().tolist()):
            got = o.cpu().numpy()
            assert c == len(w) and np.array_equal(got[:c].view(np.uint64), w) and (got[c:] == -7).all()


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("wpl", [1, 4, 16, 32])
def test_tiles_that_end_early(F, wpl, general):
    """Clauses that empty some tiles through tile literals, some through lane
    and in-word literals only, and some only through word literals, before a
    general part: counts (alone, in a batch, through a server) and models."""
    import torch
    n = 20
    rng = random.Random(7)
    text = "x19 | x18\n~x19 | x17 | ~x16\nx0 | x5\n~x0 | x6\nx3 | ~x7 | x19\n"        # tile, lane and in-word
    text += "x11 | x12 | x19\n~x12 | x11 | x18\n" + random_cnf(rng, n, 12, (2, 3))    # word bits at some tilings
    text += "x18 | ~x0 | ~x5\nx18 | x0 | ~x5\nx18 | x5 | ~x6\nx18 | x6\n~x6 | x18\n"  # nothing left where x18 is false
    if general:
        text += "(x1 ^ x2 ^ x19) | (x4 & ~x13)\n"
    p = F.Program(text, n)
    want, c = oracle.models(text, n)
    assert c > 0
    print("early", wpl, general, c, flush=True)
    assert int(F.count(p, words_per_lane=wpl).item()) == c
    assert F.count_batch([p, p], words_per_lane=wpl).cpu().tolist() == [c, c]
    sv = F.Server(2, 64, wpl)
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    t = F.program_tiles(p, wpl)
    sv.launch([p], [(0, 0, 0, t // 3), (0, 1, t // 3, t)], counts)
    torch.cuda.synchronize()
    assert sum(counts.cpu().tolist()) == c
    sv.free()
    p.set_tuning(wpl)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, [c + 1])


@pytest.mark.parametrize("first", ["tile", "low", "inword", "word", "wide"])
@pytest.mark.parametrize("wpl", [1, 8, 32])
def test_first_key_held_by_the_waves(F, wpl, first):
    """Few waves, many tiles each (one block, just under and from four tiles a
    wave on; enumerations at 2^15 tiles): clause blocks that start with a run
    of tile literals, of lane literals, of clauses with an in-word or a word
    literal in each, and with more clauses than a chunk holds."""
    rng = random.Random(wpl)
    n = 20
    tile, lane = "x19 | x18\n~x19 | x17\n~x18 | x16 | ~x17\n", "x5 | ~x7\n~x6 | x8 | x19\n"
    text = {"tile": tile + lane, "low": lane, "inword": "x0 | ~x19\nx1 | x7\n", "word": "x11 | x19\n~x11 | x7\n",
            "wide": "".join("%sx%d | %sx%d | %sx%d\n" % (rng.choice(["", "~"]), a, rng.choice(["", "~"]), b,
                                                          rng.choice(["", "~"]), c)
                            for a, b, c in (rng.sample(range(5, n), 3) for _ in range(50)))}[first]
    p = F.Program(text, n)
    want = oracle.count(text, n)
    for grid in (1, 2, F.program_tiles(p, wpl) // 16, F.program_tiles(p, wpl) // 16 + 1):
        print("first key", wpl, first, grid, want, flush=True)
        assert int(F.count(p, words_per_lane=wpl, grid_blocks=max(1, grid)).item()) == want
    if wpl == 1 and first != "low":
        n = 26  # 2^15 tiles
        text += "x25 | x24\n~x25 | x23\nx22\n~x21\nx20 | x3\n~x4\n" + "x9 & x10 & x12 & x13 & x14\n"
        q = F.Program(text, n)
        q.set_tuning(1)
        want, c = oracle.models(text, n)
        lists(lambda cap, out, tot: F.enumerate_models(q, cap, out=out, total=tot), want, [c // 2, c + 1])


def test_overlapping_enumerations(F):
    """More calls in flight than the scratch pool has blocks, on several
    streams and threads, and again after the last program has gone."""
    import threading

    import torch
    text, n = workloads.equivalence_relations(8)      # 28 letters, 4140 models
    for _ in range(2):
        p = F.Program(text, n)
        want = None
        got, errors = {}, []

        def work(t):
            try:
                s = torch.cuda.Stream()
                with torch.cuda.stream(s):
                    got[t] = [F.enumerate_models(p, 4200) for _ in range(8)]
                s.synchronize()
            except Exception as e:  # noqa: BLE001 - reported below
                errors.append(e)
        threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        for lists_ in got.values():
            for m, tot in lists_:
                assert int(tot.item()) == 4140
                m = m.cpu().numpy()[:4140]
                want = m if want is None else want
                assert np.array_equal(m, want)
        assert (np.diff(want) > 0).all()
        p.free()


@pytest.mark.parametrize("general", [False, True])
def test_more_than_2_32_tiles(F, general):
    """2^33 tiles: 44 letters at one word per lane, and a program with a general
    part over 48 letters at its own 16.  The models lie in tiles on both sides
    of the 2^32nd, several in a block of the list."""
    import itertools

    import torch
    n, low = (48, 15) if general else (44, 11)      # the tile's bits are low .. n - 1
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("the temporaries take 96 GiB")
    free = [low, low + 3, n - 1]
    text = "".join("x%d\n" % k for k in range(low, n) if k not in free)
    text += "".join("x%d\n" % k for k in range(3, low)) + "x0 | x2\n"
    if general:
        text += "(x1 ^ x%d) | (x0 & x%d)\n" % (n - 1, low)
    p = F.Program(text, n)
    if not general:
        p.set_tuning(1)
    assert F.program_tiles(p, p.info["words_per_lane"]) == 1 << 33
    want = []
    for top in itertools.product((0, 1), repeat=3):
        for x in range(8):
            if not x & 5 or (general and not ((x >> 1 & 1) ^ top[2] or (x & 1 and top[0]))):
                continue
            v = x | sum(1 << k for k in range(3, n) if k not in free) | sum(b << k for b, k in zip(top, free))
            want.append(v)
    want = np.array(sorted(want), dtype=np.uint64)
    print("2^33 tiles", n, len(want), flush=True)
    lists(lambda cap, out, tot: F.enumerate_models(p, cap, out=out, total=tot), want, [len(want) + 1])
