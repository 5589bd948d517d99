"""GPU tests of the one-kernel decode of few (sequence, KV head) units: against
the oracle, and against the stream-K kernels (which a work-split option selects)
over the forms both accept."""

import numpy as np
import pytest
import torch

import oracle

from paper_2605_20863_amd import workloads as W
from tests import _gpu_util as U

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
STREAM = {"min_blocks_per_wave": 8}  # the default split, asked for: stream-K


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2605_20863_amd import _lib
    return _lib


def wl(hq, hkv, d, kv, q_tokens=1):
    return W.Workload(f"short_{hq}_{hkv}_{d}_{kv}", 1, hq, hkv, d, "f32" if kv == "f32" else "bf16", kv,
                      ("uniform", 1, 1), cfg_id=61, q_tokens=q_tokens)


def call(lib, inp, out, **opts):
    lib.paged_decode_attention(inp.q, inp.k_cache, inp.v_cache, inp.block_table, inp.seq_lens, inp.kv_scales, out,
                               inp.softmax_scale, max_seq_len=inp.layout.max_seq_len, **opts)
    torch.cuda.synchronize()
    return out


def reference(inp):
    if inp.q.dim() == 3:
        return U.oracle_for(inp)
    w, lay = inp.workload, inp.layout
    return oracle.paged_multi_token_attention(
        q=U.raw(inp.q), k_cache=U.raw(inp.k_cache), v_cache=U.raw(inp.v_cache), block_table=lay.block_table,
        seq_lens=lay.seq_lens, softmax_scale=inp.softmax_scale, q_dtype="bf16", kv_dtype=w.kv_dtype,
        kv_scales=U.raw(inp.kv_scales) if inp.kv_scales is not None else None)


# empty and one-token sequences, the edges of a block, a pair, a group of four
# steps (64 tokens f32, 128 otherwise) and of the parts; a sequence of more than
# 32 steps a wave (the block ids' second load) alone and beside short ones
LENGTHS = {
    "edges": [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 257],
    "parts": [2000, 3, 511, 512, 513],
    "long": [9000, 40],
}
SHAPES = [("f32", 4, 4, 64, 1), ("f32", 4, 2, 128, 1), ("f32", 12, 3, 64, 1), ("f32", 14, 2, 128, 1),
          ("bf16", 8, 2, 64, 1), ("bf16", 28, 4, 128, 1), ("bf16", 16, 1, 128, 1), ("bf16", 10, 2, 128, 1),
          ("fp8_e4m3", 28, 4, 128, 1), ("fp8_e4m3", 24, 2, 64, 1),
          ("bf16", 8, 2, 128, 2), ("bf16", 28, 4, 128, 4), ("fp8_e4m3", 14, 2, 64, 3), ("fp8_e4m3", 6, 2, 128, 5)]


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("kv,hq,hkv,d,q", SHAPES)
def test_short_decode_matches_oracle_and_stream(lib, kv, hq, hkv, d, q, name):
    print(f"[short] {name} {kv} Hq={hq} Hkv={hkv} D={d} q={q}", flush=True)
    inp = W.generate(wl(hq, hkv, d, kv, q), DEV, seq_lens=LENGTHS[name])
    outs = {}
    for key, opts in (("short", {}), ("again", {}), ("stream", STREAM)):
        outs[key] = call(lib, inp, torch.full(inp.q.shape, float("nan"), dtype=torch.float32, device=DEV), **opts)
    ref = reference(inp)
    for key in ("short", "stream"):
        U.assert_close(U.out_to_f64(outs[key]), ref, kv, f"{name} {key}")
    # both sum the same products (bf16 hi + lo weights to 2^-17 of themselves, or float32) in another order
    err = (outs["short"] - outs["stream"]).norm() / outs["stream"].norm()
    assert float(err) < 1e-5, float(err)
    assert torch.equal(outs["short"], outs["again"])  # parts merge in order, whoever arrives last
    if inp.q.dtype == torch.bfloat16:
        got = call(lib, inp, torch.empty_like(inp.q))
        U.assert_close(U.out_to_f64(got), ref, kv, f"{name} bf16 out", bf16_out_rounding=True)
    assert lib.read_device_status() == 0


@pytest.mark.parametrize("kv", ["f32", "bf16"])
def test_short_decode_status_and_scale(lib, kv):
    """Clamped lengths and out-of-range blocks as in the stream-K kernels; zero
    and negative softmax scales."""
    inp = W.generate(wl(8, 2, 64, kv), DEV, seq_lens=[300, 70])
    out = torch.empty(inp.q.shape, dtype=torch.float32, device=DEV)
    lens = torch.tensor([301, -3], dtype=torch.int32, device=DEV)
    args = (inp.q, inp.k_cache, inp.v_cache, inp.block_table)
    lib.paged_decode_attention(*args, lens, inp.kv_scales, out, inp.softmax_scale, max_seq_len=300)
    assert lib.read_device_status() == lib.STATUS_LEN_CLAMPED
    U.assert_close(U.out_to_f64(out)[:1], reference(inp)[:1], kv, "clamped")
    assert not out[1].any()
    table = inp.block_table.clone()
    table[0, 3] = inp.k_cache.shape[0]
    table[0, 4] = -7
    for opts in ({}, STREAM):
        o = torch.empty_like(out)
        lib.paged_decode_attention(inp.q, inp.k_cache, inp.v_cache, table, inp.seq_lens, inp.kv_scales, o,
                                   inp.softmax_scale, max_seq_len=300, **opts)
        assert lib.read_device_status() == lib.STATUS_BAD_BLOCK
        if opts:
            assert torch.allclose(out, o, rtol=0, atol=1e-5)
        out = o
    for scale in (-0.3, 0.0):
        a, b = torch.empty_like(out), torch.empty_like(out)
        lib.paged_decode_attention(*args, inp.seq_lens, inp.kv_scales, a, scale, max_seq_len=300)
        lib.paged_decode_attention(*args, inp.seq_lens, inp.kv_scales, b, scale, max_seq_len=300, **STREAM)
        assert torch.allclose(a, b, rtol=0, atol=1e-5)


def test_short_decode_counts_are_zero_between_calls(lib):
    """Calls of other shapes, splits and kernels in between, graph replays and
    the fixed scratch: each short call finds its arrival counts at zero."""
    big = W.generate(W.SMALL_WORKLOADS["fp8kv"], DEV)
    a = W.generate(wl(28, 4, 128, "bf16"), DEV, seq_lens=[1500, 700, 2100])
    b = W.generate(wl(8, 2, 64, "f32"), DEV, seq_lens=[900, 33, 64, 2000])
    s = torch.cuda.Stream(DEV)
    want, outs = {}, {}
    for key, inp in (("a", a), ("b", b)):
        want[key] = call(lib, inp, torch.empty_like(inp.q))
        outs[key] = torch.empty_like(inp.q)
    big_out = torch.empty_like(big.q)
    with torch.cuda.stream(s):
        call(lib, big, big_out, chunks_per_wave=4, min_blocks_per_chunk=1)
        for inp, key in ((a, "a"), (b, "b")):
            call(lib, inp, outs[key])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for inp, key in ((a, "a"), (b, "b"), (a, "a")):
            lib.paged_decode_attention(inp.q, inp.k_cache, inp.v_cache, inp.block_table, inp.seq_lens, inp.kv_scales,
                                       outs[key], inp.softmax_scale, max_seq_len=inp.layout.max_seq_len)
    for r in range(4):
        with torch.cuda.stream(s):
            for o in outs.values():
                o.fill_(7.0)
            g.replay()
            call(lib, big, big_out)
        torch.cuda.synchronize()
        for key in outs:
            assert torch.equal(outs[key], want[key]), (r, key)
        for inp, key in ((a, "a"), (b, "b")):
            o = torch.empty_like(inp.q)
            lib.paged_decode_attention_noalloc(inp.q, inp.k_cache, inp.v_cache, inp.block_table, inp.seq_lens,
                                               inp.kv_scales, o, inp.softmax_scale,
                                               max_seq_len=inp.layout.max_seq_len)
            torch.cuda.synchronize()
            assert torch.equal(o, want[key]), (r, key, "fixed scratch")
    assert lib.read_device_status() == 0


def test_short_decode_after_overlapping_calls(lib):
    """Two graphs captured on one stream, replayed on two others beside eager
    calls on it: the three work in one workspace, so what they write meanwhile is
    undefined, but every later call that overlaps nothing is right again."""
    a = W.generate(wl(28, 4, 128, "bf16"), DEV, seq_lens=[1500, 700, 2100])
    b = W.generate(wl(8, 2, 64, "f32"), DEV, seq_lens=[900, 33, 64, 2000])
    s, s1, s2 = (torch.cuda.Stream(DEV) for _ in range(3))
    want, outs, graphs = {}, {}, {}
    for key, inp in (("a", a), ("b", b)):
        want[key] = call(lib, inp, torch.empty_like(inp.q))
        outs[key] = torch.empty_like(inp.q)
        with torch.cuda.stream(s):
            call(lib, inp, outs[key])
        graphs[key] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graphs[key], stream=s):
            for _ in range(8):
                lib.paged_decode_attention(inp.q, inp.k_cache, inp.v_cache, inp.block_table, inp.seq_lens,
                                           inp.kv_scales, outs[key], inp.softmax_scale,
                                           max_seq_len=inp.layout.max_seq_len)
    for r in range(5):
        print(f"[short] overlap {r}", flush=True)
        for _ in range(4):
            with torch.cuda.stream(s1):
                graphs["a"].replay()
            with torch.cuda.stream(s2):
                graphs["b"].replay()
            with torch.cuda.stream(s):
                lib.paged_decode_attention(a.q, a.k_cache, a.v_cache, a.block_table, a.seq_lens, a.kv_scales,
                                           torch.empty_like(a.q), a.softmax_scale, max_seq_len=a.layout.max_seq_len)
        torch.cuda.synchronize()
        for key, inp in (("a", a), ("b", b)):
            with torch.cuda.stream(s):
                got = call(lib, inp, torch.full_like(inp.q, 7.0))
                assert torch.equal(got, want[key]), (r, key, "eager")
                outs[key].fill_(7.0)
                graphs[key].replay()
            torch.cuda.synchronize()
            assert torch.equal(outs[key], want[key]), (r, key, "graph")
    assert lib.read_device_status() == 0


def test_short_decode_most_units(lib):
    """As many units as the header has counts for, each of one or two parts."""
    rng = np.random.default_rng(5)
    inp = W.generate(wl(16, 4, 64, "bf16"), DEV, seq_lens=rng.integers(1, 500, 48))
    out = call(lib, inp, torch.empty(inp.q.shape, dtype=torch.float32, device=DEV))
    U.assert_close(U.out_to_f64(out), reference(inp), "bf16", "192 units")
    assert lib.read_device_status() == 0
