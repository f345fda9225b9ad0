"""The short-loop and few-pixel conv kernels retire every LDS read they issue
themselves before its registers are touched, and use no scratch (their waits
count vector-memory operations); checked on the gfx950 assembly, no GPU."""
import re

import pytest

import lds_hazards as H
import test_lds_async_reads as A


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    sources = ["conv_flow.hip", "conv_flow_fused.hip", "conv_small.hip"]
    keep = A._SOURCES, dict(A._ASM)
    A._SOURCES = sources
    A._ASM.clear()
    try:
        return {s: A._asm(s, tmp_path_factory) for s in sources}
    finally:
        A._SOURCES = keep[0]
        A._ASM.clear()
        A._ASM.update(keep[1])


@A.needs_hipcc
@pytest.mark.parametrize("src", ["conv_flow.hip", "conv_flow_fused.hip", "conv_small.hip"])
def test_reads_retired_and_no_scratch(src, asm):
    ks = H.kernels(asm[src])
    assert len(ks) > 0
    bad = {name: H.hazards(lines) for name, lines in ks.items()}
    bad = {k: v for k, v in bad.items() if v}
    assert not bad, {k[:80]: sorted(v.items())[:3] for k, v in bad.items()}
    sizes = [int(v) for v in re.findall(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", asm[src])]
    assert len(sizes) >= len(ks) and not any(sizes)
