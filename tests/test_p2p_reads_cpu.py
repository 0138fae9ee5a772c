"""A property of the compiled FP32 near-field kernels with octupoles: a pair's
LDS reads are all issued before the first of them is waited for."""
import importlib.util
import os
import re
import subprocess

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_12351_amd")


def _build():
    spec = importlib.util.spec_from_file_location("fmm_build", os.path.join(PKG, "build.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_octupole_pairs_wait_for_lds_once(tmp_path):
    b = _build()
    out = str(tmp_path / "p2p_oct.s")
    subprocess.run([b.HIPCC, "-x", "hip", "--cuda-device-only", "-S", os.path.join(b.CSRC, "p2p_oct.hip"), "-o", out]
                   + b.COMMON, check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    kernels = re.findall(r"^_Z14p2p_f32_kernelILi(\d+)ELb([01])E\S*:(.*?)^\.Lfunc_end", text, re.S | re.M)
    assert len(kernels) == 16                  # masks 8-15, with the gradient and without
    for mask, grad, body in kernels:
        loops = [blk for blk in re.split(r"^\.LBB\S+:", body, flags=re.M) if "v_rsq_f32" in blk]
        assert len(loops) >= 2, (mask, grad)   # with the test for the target itself and without
        for blk in loops:
            ops = re.findall(r"^\s+(ds_read|s_waitcnt\s.*lgkmcnt)", blk, re.M)
            waits = [k for k, o in enumerate(ops) if o != "ds_read"]
            assert waits and "ds_read" in ops and "ds_read" not in ops[waits[0]:], (mask, grad, ops)
