"""Properties that the generated matrix-core M2L sources have to have, whatever
sizes and order their LDS arrays have."""
import importlib.util
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_12351_amd", "csrc")


def _load(path):
    spec = importlib.util.spec_from_file_location(os.path.basename(path)[:-3], path)
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def _gen():
    return _load(os.path.join(CSRC, "gen_m2l.py"))


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


@pytest.mark.parametrize("s", range(4))
def test_no_spills_in_the_entry_loop(tmp_path, s):
    """A register reloaded from scratch memory in the loop over the entries
    waits for all row copies under way, so none is."""
    gen, build = _gen(), _load(os.path.join(os.path.dirname(CSRC), "build.py"))
    src, out = tmp_path / "m2l.hip", tmp_path / "m2l.s"
    src.write_text(gen.gen_file(s, True, None, True, True))
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(out)] + build.COMMON,
                   check=True, capture_output=True)
    kernels = re.findall(r"^_Z\d+(m2l_p\d+_s\d_f32_hm)\w*:(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(kernels) == gen.P_MAX - s
    for name, body in kernels:
        loops = [b for b in re.split(r"^\.LBB\S+:", body, flags=re.M) if "v_mfma" in b]
        assert loops and not any("scratch_" in b for b in loops), name
