"""What a prefill call launches and where its workspace goes, on the host code
over a note-taking HIP runtime: the rule of the image, and the fallbacks of a
capture without room and of a failed allocation."""

import pytest

from paper_2605_20863_amd import _lib
from tests import _host_sim

BF16, FP8 = _lib.BF16, _lib.FP8_E4M3


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    return _host_sim.build(str(tmp_path_factory.mktemp("sim") / "libpda_sim.so"))


@pytest.fixture(autouse=True)
def fresh(sim, monkeypatch):
    for name in ("PDA_PREFILL_IMAGE_MIN_TILES", "PDA_PREFILL_IMAGE_MAX_MB"):
        monkeypatch.delenv(name, raising=False)
    sim.reset()
    sim.release()


@pytest.mark.parametrize("B,tokens,kv,image,mixed", [
    # tiles of 64 tokens (32 query, 8 KV heads); every sequence alike
    (8, 8 * 64 * 4, BF16, False, 0), (8, 8 * 64 * 5, BF16, True, 0),
    (8, 8 * 64 * 7, FP8, False, 0), (8, 8 * 64 * 8, FP8, True, 0),
    # one prompt beside rows or empty slots: no longer decided by their number
    (1, 8192, BF16, True, 0), (32, 8192 + 31, BF16, True, 5), (32, 8192, FP8, True, 8), (500, 8192 + 499, BF16, True, 5),
    # too few tiles for the second launch to pay
    (32, 6000, BF16, False, 0), (64, 64 * 64, FP8, False, 0)])
def test_image_rule(sim, B, tokens, kv, image, mixed):
    rc, n = sim.prefill(B, tokens, 32, 8, 128, kv, 512)  # up to 8,192 keys
    assert rc == 0 and bool(n["v_img"]) == image and n["img_tiles"] == mixed
    assert bool(n["k_img"]) == (image and kv == FP8)


@pytest.mark.parametrize("tiles,kv,blocks,image", [
    (9, BF16, 64, False), (10, BF16, 64, True), (9, BF16, 65, True), (12, FP8, 64, False), (13, FP8, 64, True),
    (12, FP8, 65, True)])
def test_image_rule_of_short_sequences(sim, tiles, kv, blocks, image):
    rc, n = sim.prefill(16, 16 * 64 * tiles, 32, 8, 128, kv, blocks)
    assert rc == 0 and bool(n["v_img"]) == image and n["img_tiles"] == 0  # and none is mixed


CALL = dict(B=4, T=4 * 700, hq=28, hkv=4, d=128, kv=BF16, blocks=2048)
MIXED = dict(B=40, T=6000, hq=28, hkv=4, d=128, kv=FP8, blocks=256)


@pytest.mark.parametrize("call", [CALL, MIXED], ids=["image", "mixed"])
def test_a_failed_allocation_goes_without(sim, call):
    """First without the image, then without the split; then it is an error."""
    rc, n = sim.prefill(**call)
    assert rc == 0 and n["v_img"] and n["slots"] > 0
    whole = sim.allocated()
    limit, seen = whole - 1, []
    for _ in range(3):
        sim.release()
        sim.reset(limit=limit)
        rc, n = sim.prefill(**call)
        seen.append((rc, bool(rc == 0 and n["v_img"]), bool(rc == 0 and n["slots"])))
        if rc == 0:
            assert n["img_tiles"] == 0  # without the image nothing is mixed
            limit = sim.allocated() - 1
    assert seen == [(0, False, True), (0, False, False), (_lib.ENOMEM, False, False)]


@pytest.mark.parametrize("call", [CALL, MIXED], ids=["image", "mixed"])
def test_a_capture_without_room_goes_without(sim, monkeypatch, call):
    """The workspace's room decides: partials first, then the image. A capture
    that has none for the work list is refused."""
    rc, n = sim.prefill(**call)
    assert rc == 0 and n["v_img"] and n["slots"] > 0
    sim.reset(capture=5)
    rc, n = sim.prefill(**call)  # sized by the eager call: all of it
    assert rc == 0 and n["v_img"] and n["slots"] > 0
    sim.reset()
    sim.release()
    monkeypatch.setenv("PDA_PREFILL_IMAGE_MAX_MB", "0")
    assert sim.prefill(**call)[0] == 0  # room for the partials, not for the image
    monkeypatch.delenv("PDA_PREFILL_IMAGE_MAX_MB")
    sim.reset(capture=6)
    rc, n = sim.prefill(**call)
    assert rc == 0 and not n["v_img"] and n["slots"] > 0 and n["img_tiles"] == 0
    sim.reset()
    sim.release()
    assert sim.prefill(**{**call, "blocks": 16})[0] == 0  # short tables: no split, room for a list
    monkeypatch.setenv("PDA_PREFILL_IMAGE_MAX_MB", "0")
    sim.reset()
    sim.release()
    assert sim.prefill(**{**call, "blocks": 16})[0] == 0
    sim.reset(capture=7)
    rc, n = sim.prefill(**call)
    assert rc == 0 and not n["v_img"] and n["slots"] == 0
    sim.reset()
    sim.release()
    sim.reset(capture=8)
    assert sim.prefill(**call)[0] == _lib.EINVAL


def test_nothing_overlaps_in_the_workspace(sim):
    """Lists, parts, splits, partials and image, in order and inside the allocation."""
    for call in (CALL, MIXED, {**CALL, "kv": FP8}, {**MIXED, "B": 1200, "T": 20000, "blocks": 65}):
        sim.release()
        rc, n = sim.prefill(**call)
        assert rc == 0 and n["v_img"]
        lists = 2 if n["img_tiles"] else 1
        cols = n["slots"] * call["hkv"] * 256
        assert n["items"] >= n["hdr"] + 4 * 32
        assert n["parts"] >= n["items"] + lists * n["list_max"] * 16
        end = n["parts"]
        if n["slots"]:
            assert n["splits"] >= n["parts"] + lists * n["list_max"] * 16
            assert n["part_ml"] >= n["splits"] + n["slots"] // 2 * 16
            assert n["part_acc"] >= n["part_ml"] + cols * 8
            end = n["part_acc"] + cols * 4 * call["d"]
        img = (call["B"] * call["blocks"] + 1) * call["hkv"] * 16 * call["d"] * 2
        assert n["v_img"] >= end
        last = n["v_img"] + img
        if call["kv"] == FP8:
            assert n["k_img"] >= last
            last = n["k_img"] + img
        assert sim.room(last) >= 0
