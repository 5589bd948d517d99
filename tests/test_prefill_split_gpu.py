"""GPU tests of the prefill call's split plan (few query tiles over long caches:
each tile's keys are split over several work items whose partials a merge
kernel combines) and of the rule that leaves out the image where few tiles
would read it, against the oracle."""

import numpy as np
import pytest
import torch

from paper_2605_20863_amd import workloads as W
from tests import _gpu_util as U
from tests.test_prefill_gpu import DEV, GROUPS, check, lib, run, wl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["image", "staging"])
def path(request, monkeypatch):
    """The tile source whatever the number of tiles: the image always, or never."""
    monkeypatch.setenv("PDA_PREFILL_IMAGE_MIN_TILES", "0")
    if request.param == "staging":
        monkeypatch.setenv("PDA_PREFILL_IMAGE_MAX_MB", "0")
    else:
        monkeypatch.delenv("PDA_PREFILL_IMAGE_MAX_MB", raising=False)
    return request.param


# (lengths, query tokens): chunks over caches long enough to split (items of at
# least 16 pairs of 32 keys) -- one sequence alone; lengths around multiples of
# a pair, a block and an item's four pairs; a long sequence among short and
# empty ones, with more queries than keys in one
# -- and, for the plan's list of tiles, runs of sequences without queries first,
# last and between others, and as many sequences as it takes
SPLITS = {
    "alone": ([5000], [70]),
    "one_token": ([3333], [1]),
    "edges": ([2047, 2048, 2049, 1024, 1025, 544, 513, 31], [5, 64, 33, 40, 17, 32, 1, 31]),
    "mixed": ([6000, 0, 20, 1, 300, 48, 5], [90, 0, 20, 1, 200, 16, 9]),
    "without_queries": ([100, 40, 3000, 0, 9, 700, 700, 5, 60], [0, 0, 150, 0, 0, 90, 300, 0, 0]),
    "most_sequences": ([700] + [17 + i % 30 for i in range(1023)], [60] + [i % 3 for i in range(1023)]),
}


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (6, 2, 64), (16, 1, 128), (15, 5, 64)])
@pytest.mark.parametrize("name", list(SPLITS))
def test_prefill_split_matches_oracle(lib, path, kv, hq, hkv, d, name):
    lens, counts = SPLITS[name]
    print(f"[prefill split] {name} {path} kv={kv} Hq={hq} Hkv={hkv} D={d}", flush=True)
    pin = W.generate_prefill(wl(hq, hkv, d, kv), DEV, seq_lens=lens, q_counts=counts)
    check(lib, pin, f"{name} {path}")
    a, b = run(lib, pin, torch.bfloat16), run(lib, pin, torch.bfloat16)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))  # the merge runs in item order


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
def test_prefill_split_paths_agree_bitwise(lib, monkeypatch, kv):
    """The plan does not depend on where the tiles come from."""
    pin = W.generate_prefill(wl(28, 4, 128, kv), DEV, seq_lens=[4000, 700, 90], q_counts=[40, 64, 90])
    outs = []
    for mb in ("8192", "0"):
        monkeypatch.setenv("PDA_PREFILL_IMAGE_MIN_TILES", "0")
        monkeypatch.setenv("PDA_PREFILL_IMAGE_MAX_MB", mb)
        outs.append(run(lib, pin, torch.float32))
    monkeypatch.delenv("PDA_PREFILL_IMAGE_MIN_TILES")
    outs.append(run(lib, pin, torch.float32))  # the default rule: too few tiles for the image
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    assert torch.equal(outs[0].view(torch.int32), outs[2].view(torch.int32))


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", GROUPS)
def test_prefill_forced_image_matches_oracle(lib, monkeypatch, kv, d, hq, hkv):
    """The image path at every group size, for batches whose few tiles would
    not choose it."""
    monkeypatch.setenv("PDA_PREFILL_IMAGE_MIN_TILES", "0")
    monkeypatch.delenv("PDA_PREFILL_IMAGE_MAX_MB", raising=False)
    pin = W.generate_prefill(wl(hq, hkv, d, kv), DEV, seq_lens=[1, 15, 16, 17, 33, 100, 257, 700],
                             q_counts=[1, 15, 16, 5, 33, 64, 257, 300])
    check(lib, pin, f"image {kv} D{d} G{hq // hkv}")


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
def test_prefill_more_units_than_the_split_takes(lib, kv):
    """Above the split's bound on units the queues alone spread the tiles."""
    rng = np.random.default_rng(3)
    lens = rng.integers(1, 260, 400)
    pin = W.generate_prefill(wl(16, 16, 64, kv), DEV, seq_lens=lens, q_counts=np.maximum(lens // 2, 1))
    out = run(lib, pin, torch.float32)
    U.assert_close(U.out_to_f64(out), U.oracle_prefill_whole(pin, "units"), kv, f"units {kv}")
    assert lib.read_device_status() == 0
