"""GPU tests of mixed prefill calls: long prompts beside sequences of few query
tiles (one-token rows, empty slots), where the plan writes the image for the
former only and a second attention launch reads the latter from the cache. The
same bits as with every sequence's tiles from the image, or from the cache."""

import numpy as np
import pytest
import torch

from paper_2605_20863_amd import workloads as W
from tests import _gpu_util as U
from tests.test_prefill_gpu import DEV, lib, run, wl  # noqa: F401

pytestmark = pytest.mark.gpu

# 16 query heads per KV head: tiles of 16 tokens, so 100 tiles (the least of a
# mixed call) are 1,600 tokens. Sequences of as many tiles as the image takes
# (5 bf16, 8 fp8) and one fewer; rows over long and short caches; empty slots.
LENS = [1500, 600, 900, 128, 80, 112, 64, 0, 33] + [700, 1, 16, 17, 300, 0] * 6
COUNTS = [1500, 200, 0, 128, 80, 112, 64, 0, 3] + [1, 1, 1, 0, 1, 0] * 6


def outputs(lib, pin, monkeypatch, dtype=torch.float32):  # noqa: F811
    out = {}
    for key, env in (("mixed", {}), ("image", {"PDA_PREFILL_IMAGE_MIN_TILES": "0"}),
                     ("cache", {"PDA_PREFILL_IMAGE_MAX_MB": "0"})):
        for name in ("PDA_PREFILL_IMAGE_MIN_TILES", "PDA_PREFILL_IMAGE_MAX_MB"):
            monkeypatch.delenv(name, raising=False)
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        out[key] = run(lib, pin, dtype)
    return out


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("plan", ["split", "whole"])
@pytest.mark.parametrize("hq,hkv,d", [(16, 1, 128), (48, 3, 64)])
def test_mixed_matches_oracle_and_both_paths(lib, monkeypatch, kv, plan, hq, hkv, d):  # noqa: F811
    lens, counts = list(LENS), list(COUNTS)
    if plan == "whole":  # more sequences than the split plan takes
        lens += [1 + i % 20 for i in range(1100)]
        counts += [i % 2 for i in range(1100)]
    print(f"[prefill mixed] {plan} kv={kv} Hq={hq} Hkv={hkv} D={d}", flush=True)
    pin = W.generate_prefill(wl(hq, hkv, d, kv), DEV, seq_lens=lens, q_counts=counts)
    tiles = sum(counts) // 16
    assert 100 <= tiles < 5 * len(lens)
    got = outputs(lib, pin, monkeypatch)
    for key in ("image", "cache"):
        assert torch.equal(got["mixed"].view(torch.int32), got[key].view(torch.int32)), key
    U.assert_close(U.out_to_f64(got["mixed"]), U.oracle_prefill_whole(pin, f"mixed {plan}"), kv, f"mixed {plan} {kv}")
    assert lib.read_device_status() == 0


@pytest.mark.parametrize("seq", [0, 9], ids=["imaged", "row"])
def test_mixed_status_bits(lib, seq):  # noqa: F811
    """A value outside the fp16 range, and a block id out of range, in a prompt
    and in a row: the second launch's status counts as the first's does."""
    pin = W.generate_prefill(wl(16, 1, 64, "bf16"), DEV, seq_lens=LENS, q_counts=COUNTS)
    c = pin.cache
    block = int(c.layout.block_table[seq, 0])
    keep = c.v_cache[block, 0, 5, 2].clone()
    c.v_cache[block, 0, 5, 2] = 1e6
    run(lib, pin, torch.float32)
    assert lib.read_device_status() == lib.STATUS_HALF_RANGE
    assert lib.read_device_status() == 0
    c.v_cache[block, 0, 5, 2] = keep
    for bad in (c.k_cache.shape[0], -2):
        c.block_table[seq, 1] = bad
        run(lib, pin, torch.float32)
        assert lib.read_device_status() == lib.STATUS_BAD_BLOCK
    c.block_table[seq, 1] = int(c.layout.block_table[seq, 1])
    pin.q_offsets[5] = pin.q_offsets[4] - 1  # decreasing
    run(lib, pin, torch.float32)
    assert lib.read_device_status() == lib.STATUS_BAD_OFFSETS


def test_mixed_graph_replays(lib):  # noqa: F811
    """Captured with room for both lists and the image, and replayed with other
    queries and lengths in place."""
    pin = W.generate_prefill(wl(16, 1, 128, "bf16"), DEV, seq_lens=LENS, q_counts=COUNTS)
    c = pin.cache
    out_g, out_e = (torch.empty(pin.q.shape, dtype=torch.float32, device=DEV) for _ in range(2))

    def call(out):
        lib.paged_prefill_attention(pin.q, pin.q_offsets, c.k_cache, c.v_cache, c.block_table, c.seq_lens, None, out,
                                    c.softmax_scale, max_seq_len=c.layout.max_seq_len)

    s = torch.cuda.Stream(DEV)
    with torch.cuda.stream(s):
        call(out_e)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call(out_g)
    rng = np.random.default_rng(3)
    for r in range(4):
        with torch.cuda.stream(s):
            pin.q.copy_(torch.randn(pin.q.shape, device=DEV).to(pin.q.dtype))
            c.seq_lens.copy_(torch.from_numpy(np.maximum(np.array(LENS) - rng.integers(0, 9, len(LENS)), 0).astype(np.int32)))
            g.replay()
            call(out_e)
        torch.cuda.synchronize()
        print(f"[prefill mixed] replay {r}", flush=True)
        assert torch.equal(out_g.view(torch.int32), out_e.view(torch.int32)), r
    assert lib.read_device_status() == 0
