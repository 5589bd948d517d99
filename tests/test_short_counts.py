"""The short decode's arrival counts (which workgroup of a unit merges its
parts) must not depend on what earlier calls left in them: calls that overlapped
on one workspace spoil each other, but never a later call. The host side runs
over a note-taking HIP runtime; the device side is a line-for-line model of the
count, run over random interleavings of overlapping calls."""

import numpy as np
import pytest

from paper_2605_20863_amd import _lib
from tests import _host_sim

BITS = 16  # kShortCountBits
COUNT_BYTES = 2 * 192 * 128  # kShortCountBytes


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    return _host_sim.build(str(tmp_path_factory.mktemp("sim") / "libpda_sim.so"))


def arrive(words, u, epoch, parts):
    """One workgroup's arrival; True for the one that merges."""
    none = epoch << BITS
    words[u] = max(words[u], none)
    before = words[u]
    words[u] += 1
    last = before == none + parts - 1
    if last:
        words[u] -= parts
    return last


@pytest.mark.parametrize("seed", range(50))
def test_a_call_alone_merges_once_whatever_overlapped_before(seed):
    rng = np.random.default_rng(seed)
    words, epoch = [0], 0
    for _ in range(20):
        # some calls on one unit, their arrivals interleaved at random
        calls = []
        for _ in range(int(rng.integers(1, 4))):
            epoch += 1
            calls.append((epoch, int(rng.integers(2, 33))))
        order = np.repeat(np.arange(len(calls)), [p for _, p in calls])
        rng.shuffle(order)
        for i in order:
            arrive(words, 0, *calls[i])
        epoch += 1  # now one alone
        parts = int(rng.integers(2, 33))
        assert [arrive(words, 0, epoch, parts) for _ in range(parts)] == [False] * (parts - 1) + [True]
    # a graph's words: cleared where it first uses them, back at zero after each call
    words[0] = 0
    for parts in (2, 7, 32, 3):
        assert [arrive(words, 0, 0, parts) for _ in range(parts)] == [False] * (parts - 1) + [True]
        assert words[0] == 0


SHORT = dict(B=4, hq=28, hkv=4, d=128, kv=_lib.BF16, blocks=64)


def test_every_eager_call_counts_from_an_epoch_of_its_own(sim):
    sim.release()
    sim.reset()
    seen = set()
    for i in range(6):
        # calls of other sizes and kernels in between, growth of the workspace among them
        rc, n = sim.decode(**{**SHORT, "B": 1 + i % 3})
        assert rc == 0 and n["parts"] > 1 and n["clear"] == 0
        assert n["epoch"] > 0 and n["epoch"] not in seen
        seen.add(n["epoch"])
        assert sim.lib.sim_room(n["hdr"] - COUNT_BYTES) > COUNT_BYTES  # right before the header, inside the allocation
        assert sim.decode(**{**SHORT, "B": 64 << i})[1]["parts"] == 0
    # another stream has a workspace and epochs of its own
    rc, other = sim.decode(**SHORT, stream=0x2000)
    assert rc == 0 and other["hdr"] != n["hdr"]


def test_a_graph_clears_its_counts_once(sim):
    sim.release()
    sim.reset()
    rc, eager = sim.decode(**SHORT)
    assert rc == 0
    for capture in (7, 9):
        sim.reset(capture=capture)
        for i in range(3):
            rc, n = sim.decode(**SHORT)
            assert rc == 0 and n["parts"] > 1 and n["epoch"] == 0
            assert n["clear"] == (i == 0), "the first call of a capture clears, the others find zero"
    sim.reset()
    rc, n = sim.decode(**SHORT)
    assert rc == 0 and n["epoch"] > eager["epoch"] and n["clear"] == 0


def test_the_fixed_scratch_clears_at_every_call(sim):
    sim.reset()
    for capture in (0, 0, 3, 3):
        sim.reset(capture=capture)
        rc, n = sim.decode(**SHORT, noalloc=True)
        assert rc == 0 and n["parts"] > 1 and n["clear"] == 1 and n["epoch"] == 0


@pytest.mark.parametrize("kv,units,tokens,short", [
    # (sequence, KV head) units of 4 KV heads; 2 parts each at 96: the longest a wave may run
    (_lib.BF16, 96, 9 * 256, True), (_lib.BF16, 96, 9 * 256 + 16, False), (_lib.BF16, 96, 3184, False),
    (_lib.FP8_E4M3, 96, 3184, True), (_lib.BF16, 80, 4576, False), (_lib.BF16, 64, 6144, True), (_lib.BF16, 128, 1792, True),
    # one unit a sequence and head of few: up to the bound on units times length
    (_lib.BF16, 4, 98304, True), (_lib.BF16, 4, 98304 + 16, False), (_lib.BF16, 192, 784, True), (_lib.BF16, 196, 64, False)])
def test_short_decode_rule(sim, kv, units, tokens, short):
    sim.reset()
    rc, n = sim.decode(units // 4, 28, 4, 128, kv, blocks=tokens // 16)
    assert rc == 0 and (n["parts"] > 0) == short
