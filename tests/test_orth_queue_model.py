"""Host model of how the blocks of the batched orthogonalisation take items
from their queue (orth_persistent in csrc/tsg_batched.hip).

A launch has `grid` blocks of which `resident` run at a time (other launches,
or a mask of compute units, hold the rest of the chip); a block that has left
makes room for the next one.  Slab items never wait; an update item waits for
every slab item of its instance.  A block draws an item, and the next one
before it works on it.  For every order in which running blocks can step, no
state may be reached in which work is left and every running block waits."""
import os
import random
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1905_03136_amd", "csrc",
                   "tsg_batched.hip")


def build_queue(slabs, pieces, lag):
    """[(phase, instance)]: the updates of rank r come after the slabs of ranks up to r + lag."""
    n, out = len(slabs), []
    for step in range(n + lag):
        if step < n:
            out += [(1, step)] * slabs[step]
        if 0 <= step - lag < n:
            out += [(2, step - lag)] * pieces[step - lag]
    return out


def finishes(queue, slabs, grid, resident, rng, first_by_number=False):
    """Whether the launch drains; blocks step in random order."""
    head = grid if first_by_number else 0
    left = list(slabs)
    done, started = 0, 0
    running = {}

    def draw():
        nonlocal head
        head += 1
        return head - 1

    while True:
        while started < grid and len(running) < resident:  # blocks start in order
            b, started = started, started + 1
            q = b if first_by_number else draw()
            if q < len(queue):
                running[b] = [q, draw()]
        if not running:
            assert started == grid
            return done == len(queue)
        can = [b for b, (q, _) in running.items() if queue[q][0] == 1 or left[queue[q][1]] == 0]
        if not can:
            return False
        b = rng.choice(can)
        q, nxt = running.pop(b)
        phase, inst = queue[q]
        left[inst] -= phase == 1
        done += 1
        if nxt < len(queue):
            running[b] = [nxt, draw()]


@pytest.mark.parametrize("resident", [1, 2, 5, 16])
def test_any_residency_and_lag_drains(resident):
    rng = random.Random(resident)
    for trial in range(40):
        n = rng.randint(1, 9)
        slabs = [rng.randint(1, 7) for _ in range(n)]
        pieces = [rng.randint(0, 9) for _ in range(n)]
        for lag in range(1, n + 1):
            q = build_queue(slabs, pieces, lag)
            assert finishes(q, slabs, 16, resident, rng), (slabs, pieces, lag)


def test_the_model_finds_items_held_by_blocks_that_do_not_run():
    """First items bound to the blocks' numbers wait for blocks that are not running."""
    rng = random.Random(0)
    slabs, pieces = [8] * 2, [8] * 2
    q = build_queue(slabs, pieces, 2)
    assert finishes(q, slabs, 16, 16, rng, first_by_number=True)
    assert not finishes(q, slabs, 16, 4, rng, first_by_number=True)


def test_the_kernel_draws_every_item_from_the_head():
    """As the model has it: no item of the kernel depends on a block's number."""
    with open(SRC) as f:
        text = f.read()
    body = text[text.index("orth_persistent(const DevDesc"):text.index("// ---", text.index("orth_persistent(const DevDesc"))]
    assert "blockIdx" not in body
    assert re.findall(r"\bq = ([^;]*);", body) == ["__builtin_amdgcn_readfirstlane(s_q)"] * 2
    assert re.findall(r"(?:s_q|next) = draw\(\)", body) == ["s_q = draw()", "next = draw()"]
