"""Host-side checks over every public header (no GPU needed): all symbols any
of them declares are exported, each compiles by itself, and the calls of
octaoctree_render.h refuse bad input before any device work."""
import ctypes as C
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_08469_amd import binding
from test_abi_host import L, _disp, _mlp, _tree  # noqa: F401

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HEADERS = sorted(f for f in os.listdir(os.path.join(ROOT, "include")) if f.endswith(".h"))


def test_every_header_declares_only_exported_symbols(L):  # noqa: F811
    names = {}
    for h in HEADERS:
        text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", h)).read(), flags=re.S)
        for n in re.findall(r"\b(oo_\w+)\s*\(", text):
            names.setdefault(n, []).append(h)
    assert len(names) == 19 and all(len(v) == 1 for v in names.values()), names
    assert {"oo_query_workspace_bytes", "oo_query_fwd_ws"} <= set(names)
    for n in sorted(names):
        assert hasattr(L, n), n


@pytest.mark.parametrize("header", HEADERS)
def test_header_compiles_by_itself(header, tmp_path):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("needs a host C compiler and the HIP runtime headers")
    src = tmp_path / "one.c"
    src.write_text(f'#include "{header}"\nint (*f)(const oo_tree*, const oo_mlp*, int64_t, size_t*) = '
                   'oo_query_workspace_bytes;\n')
    subprocess.run([cc, "-std=c99", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROCM, "include"), "-c", str(src), "-o", str(tmp_path / "one.o")], check=True)


def _shifted(**kw):
    t = _tree(**kw)
    t.interp = 1
    t.disparity = C.pointer(_disp())
    return t


def test_query_workspace_bytes_validation(L):  # noqa: F811
    t, m, n = _shifted(), _mlp(), C.c_size_t(7)

    def size(t, m, B):
        rc = L.oo_query_workspace_bytes(C.byref(t), C.byref(m), B, C.byref(n))
        return n.value if rc == 0 else rc

    assert size(_tree(), m, 1000) == 0                  # no predictor: none needed
    assert size(t, m, 0) == 0
    assert size(t, m, 1000) >= 1000 * (4 + 24 * 2)      # a disparity and an FP16 decoder input row each
    assert size(t, m, 1 << 40) < 2 * (1 << 20) * (4 + 24 * 2)  # large batches run in passes
    assert size(t, m, -1) == -1 and b"B must" in L.oo_last_error()
    assert L.oo_query_workspace_bytes(C.byref(t), C.byref(m), 16, None) == -1 and b"bytes" in L.oo_last_error()
    assert size(t, _mlp(dtype=binding.BF16), 16) == -4  # dtype pair
    assert size(t, _mlp(K0=20), 16) == -1 and size(t, _mlp(H=96), 16) == -4
    bad = _shifted()
    bad.interp = 0
    assert size(bad, m, 16) == -1 and b"OO_INTERP_PAPER" in L.oo_last_error()


def test_query_with_workspace_validation(L):  # noqa: F811
    t, m, wide, n = _shifted(), _mlp(), _mlp(K0=24 + 16), C.c_size_t(0)
    p = C.c_void_p(0x4000)
    assert L.oo_query_workspace_bytes(C.byref(t), C.byref(m), 16, C.byref(n)) == 0

    def call(t=t, m=m, x=p, d=p, attr=None, B=16, rgb=p, ws=p, size=n.value):
        return L.oo_query_fwd_ws(C.byref(t), C.byref(m), x, d, attr, B, rgb, ws, size, None)

    assert call(B=0, x=None, d=None, rgb=None, ws=None, size=0) == 0
    assert call(B=-1) == -1 and b"B must" in L.oo_last_error()
    for k in ("x", "d", "rgb"):
        assert call(**{k: None}) == -1 and b"required" in L.oo_last_error()
    assert call(m=wide) == -1 and b"attr" in L.oo_last_error()
    assert call(m=_mlp(dtype=binding.F32)) == -4
    assert call(ws=None) == -1 and b"workspace" in L.oo_last_error()
    assert call(size=n.value - 1) == -1 and b"workspace" in L.oo_last_error()
    assert call(B=17 << 20) == -1 and b"workspace" in L.oo_last_error()
    # the kernels store whole vectors there
    assert call(ws=C.c_void_p(0x4008)) == -1 and b"16-byte aligned" in L.oo_last_error()
