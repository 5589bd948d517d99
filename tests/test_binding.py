"""The torch front end's handling of a decode call's options, on the CPU: the
tensor checks and the launch replaced, everything between as it is."""

import pytest
import torch

from paper_2605_20863_amd import _lib

OPTIONS = ["waves_per_cu", "min_blocks_per_wave", "chunks_per_wave", "min_blocks_per_chunk"]


@pytest.fixture
def call(monkeypatch):
    monkeypatch.setattr(_lib, "_check_tensors", lambda tensors: 0)
    launched = []
    monkeypatch.setattr(_lib, "_launch", lambda fn, index, stream, *args: launched.append(args[-1]))
    q = torch.zeros((1, 4, 64), dtype=torch.bfloat16)
    k, v = torch.zeros((2, 1, 16, 64), dtype=torch.bfloat16), torch.zeros((2, 1, 64, 16), dtype=torch.bfloat16)
    table, lens = torch.zeros((1, 1), dtype=torch.int32), torch.ones(1, dtype=torch.int32)

    def run(**options):
        _lib.paged_decode_attention(q, k, v, table, lens, None, torch.empty_like(q), 0.1, **options)
        return launched[-1]

    return run


@pytest.mark.parametrize("name", OPTIONS)
def test_option_values(call, name):
    assert call() is None  # the defaults
    assert call(**{name: 0}) is None
    assert getattr(call(**{name: 3}), name) == 3
    for wrong in (None, "", [], "x"):  # refused, not taken for the default
        with pytest.raises((TypeError, ValueError)):
            call(**{name: wrong})


def test_variants(call):
    assert call(variant="mfma").variant == _lib.VARIANT_MFMA
    with pytest.raises(KeyError):
        call(variant="none")
