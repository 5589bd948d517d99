"""The M0 checks of test_prefill_isa on the prefill kernels of the split plan,
which share the attention kernels' body and their direct loads. Host-only."""

import re

from tests.test_prefill_isa import kernels, prefill_asm  # noqa: F401
from tests.test_prefill_isa import test_no_other_reads_of_m0 as no_other_reads_of_m0


def test_split_kernels_m0(prefill_asm):  # noqa: F811
    asm = "\n".join(re.sub(r"^(_Z\S*)split_prefill", r"\1split_prefill_kernel", line)
                    for line in prefill_asm.splitlines())
    split = {n: ins for n, ins in kernels(asm).items() if "split" in n}
    assert len(split) == 8, sorted(split)
    for name, ins in split.items():
        m0 = [i for i, s in enumerate(ins) if re.search(r"\bm0\b", s)]
        loads = [i for i, s in enumerate(ins) if s.startswith("global_load_lds")]
        assert [i + 1 for i in m0] == loads and all(ins[i].startswith("s_mov_b32 m0, ") for i in m0), name
    assert sum(any(s.startswith("global_load_lds") for s in ins) for ins in split.values()) == 4
    no_other_reads_of_m0(asm)


def test_split_kernels_spill_nothing(prefill_asm):  # noqa: F811
    """A part's slot and first key stay out of the registers of the pair loop."""
    asm = "\n".join(re.sub(r"^(_Z\S*)split_prefill", r"\1split_prefill_kernel", line)
                    for line in prefill_asm.splitlines())
    for name, ins in kernels(asm).items():
        assert not any(s.startswith(("scratch_", "buffer_store", "buffer_load")) for s in ins), name
