"""The binding without its native call path, which is built against one torch for ROCm: everything goes through the Python code then."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2503_14985_amd")
SCRIPT = """
import sys, types, torch
%s
from paper_2503_14985_amd import binding as b
assert b.mlt_version() and b.mlt_query_tiling(0, (16, 4096, 4096, 1), 0)
assert (b._fast.__name__ == "paper_2503_14985_amd._fastcall") == %r
t = torch.zeros(2, 2, dtype=torch.bfloat16)
for call in (lambda: b.mlt_gemm(t, t, C=t), lambda: b.mlt_gemm_acc(t, t, t.float()), lambda: b.mlt_gemm_bias_act(t, t, C=t),
             lambda: b.mlt_mha_fwd(*[t.reshape(1, 1, 2, 2)] * 3, 1.0, O=t.reshape(1, 1, 2, 2)),
             lambda: b.mlt_paged_attn_decode(t.reshape(1, 2, 2), *[t.reshape(1, 2, 1, 2)] * 2, torch.zeros(1, 1, dtype=torch.int32), torch.ones(1, dtype=torch.int32), 1.0)):
    try:
        call()
    except ValueError as e:
        assert "GPU" in str(e), e
    else:
        raise AssertionError("CPU tensors were taken")
print("ok")
"""


@pytest.mark.parametrize("fastcall,torch_version,native", [("built", None, True), (None, None, False), ("broken", None, False), ("built", "9.9.9+rocm9", False)])
def test_binding_with_and_without_the_native_call_path(tmp_path, fastcall, torch_version, native):
    import torch
    if torch.version.hip is None or not os.path.exists(os.path.join(PKG, "_fastcall.so")):
        if fastcall == "built":
            pytest.skip("no native call path is built here")
    pkg = tmp_path / "paper_2503_14985_amd"
    pkg.mkdir()
    for f in os.listdir(PKG):
        if f.endswith(".py"):
            shutil.copy(os.path.join(PKG, f), pkg / f)
    os.symlink(os.path.join(PKG, "libmlt.so"), pkg / "libmlt.so")
    if fastcall == "built":
        os.symlink(os.path.join(PKG, "_fastcall.so"), pkg / "_fastcall.so")
    elif fastcall == "broken":
        (pkg / "_fastcall.so").write_bytes(b"not a library")
    script = SCRIPT % ("torch.__version__ = %r" % torch_version if torch_version else "", native)
    r = subprocess.run([sys.executable, "-c", script], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
