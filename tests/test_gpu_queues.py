"""The work queues of the batch kernels: every item is taken once, whether by
number, popped or popped from another queue, for grids that fill the eight
queues evenly or not, with fewer and with more items than takers."""

import random

import pytest

import oracle
from formula_gen import random_cnf, random_program

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1310_6978_amd import fbg
    return fbg


@pytest.mark.parametrize("cofactor", [False, True])
@pytest.mark.parametrize("np_", [1, 3, 9, 50])
def test_every_item_once(F, np_, cofactor):
    rng = random.Random(np_)
    texts = []
    for i in range(np_):
        n = rng.choice([6, 11, 14, 17])
        text = random_cnf(rng, n, 2 * n, (2, 4)) if i % 3 else random_program(rng, n)[1]
        if cofactor and n >= 14:                # (most tiles dead, else it is set aside)
            text = "x%d\nx%d\n" % (n - 1, n - 2) + text
        texts.append((text, n))
    progs = [F.Program(t, n) for t, n in texts]
    want = [oracle.count(t, n) for t, n in texts]
    for wpl in (1, 16):
        for grid in (0, 1, 3, 7, 8, 9, 17, 64):
            print("queues", np_, cofactor, wpl, grid, flush=True)
            b = F.Batch(progs, words_per_lane=wpl, grid_blocks=grid, cofactor=cofactor)
            for _ in range(2):
                assert b.count().cpu().tolist() == want
            assert b.count(graph=True).cpu().tolist() == want
            b.free()


@pytest.mark.parametrize("np_,n", [(1, 20), (1, 22), (4, 18), (4, 22), (40, 17)])
def test_clause_plans_on_both_sides_of_the_pops(F, np_, n):
    """A grid of 8 blocks: short items, one for each wave, then long ones, popped."""
    rng = random.Random(7 * n + np_)
    texts = [(random_cnf(rng, n - i % 3, 4 * n, (3, 3)), n - i % 3) for i in range(np_)]
    progs = [F.Program(t, m) for t, m in texts]
    want = [oracle.count(t, m) for t, m in texts]
    for wpl in (1, 4):
        print("clause plans", np_, n, wpl, flush=True)
        b = F.Batch(progs, words_per_lane=wpl, grid_blocks=8)
        for _ in range(2):
            assert b.count().cpu().tolist() == want
        b.free()
