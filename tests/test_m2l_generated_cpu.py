"""Properties that the generated matrix-core M2L sources have to have, whatever
sizes and order their LDS arrays have."""
import importlib.util
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_12351_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen_m2l", os.path.join(CSRC, "gen_m2l.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_staged_rows_start_at_a_line():
    """A lane reads quad q of its staged row at its row's address with 16 q
    exclusive-or'ed in, q < 8: right only where rows start at multiples of 128
    bytes, so every array of staged rows asks for that alignment itself."""
    gen = _gen()
    kernels = 0
    for s in range(4):
        for p in range(s + 1, gen.P_MAX + 1):
            src = gen.gen_kernel_mfma(p, s)[0]
            arrays = re.findall(r"__shared__ (alignas\((\d+)\) )?float4 area\[(\d+)\]", src)
            assert len(arrays) == 1, (p, s)
            flips = max(int(v) for v in re.findall(r"\^ (\d+)u\)", src))
            assert arrays[0][0] and int(arrays[0][1]) % 128 == 0 and flips < int(arrays[0][1]), (p, s)
            kernels += 1
    assert kernels == 34
