"""The native side of a call: plain tensors by their C++ object, everything else as the Python function decides."""
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402
import paper_2001_00532_amd.binding as binding  # noqa: E402


class Sub(torch.Tensor):
    pass


def test_what_is_not_plain_is_refused_as_before():
    psk.lib()
    assert binding._ptr is not binding._ptr_checked and binding._ptr(None) is None
    f = torch.zeros(4)
    i = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(ValueError, match="device tensor"):
        binding._ptr(f)
    with pytest.raises(ValueError, match="device tensor"):
        binding._ptr(f.as_subclass(Sub), torch.float32)
    with pytest.raises(AttributeError):
        binding._ptr(7)
    with pytest.raises(ValueError, match="device tensor"):
        psk.psk_spmv_csr(1, 1, 1, i, i, f, f, f, ws=f)
    with pytest.raises((TypeError, ValueError)):
        psk.psk_spmv_csr("a", 1, 1, i, i, f, f, f, ws=f)


WITHOUT = """
import sys, types, warnings
import torch
{prepare}
import paper_2001_00532_amd as psk, paper_2001_00532_amd.binding as binding
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    psk.lib()
assert len(seen) == 1 and {words!r} in str(seen[0].message), [str(w.message) for w in seen]
assert binding._marshal is None and binding._ptr is binding._ptr_checked
assert psk.psk_default_tile(psk.PSK_OP_SPMV_CSR) > 0
if torch.cuda.is_available():
    for dtype, f, op in ((torch.float32, psk.psk_spmv_csr, psk.PSK_OP_SPMV_CSR), (torch.float64, psk.psk_spmv_csr_f64, psk.PSK_OP_SPMV_CSR_F64)):
        i = lambda *a: torch.tensor(a, dtype=torch.int32, device="cuda")
        v = lambda *a: torch.tensor(a, dtype=dtype, device="cuda")
        y = f(3, 3, 3, i(0, 2, 2, 3), i(0, 2, 1), v(1, 2, 3), v(1, 10, 100), torch.empty(3, dtype=dtype, device="cuda"), ws=psk.workspace(op, 3, 3))
        assert y.cpu().tolist() == [201, 0, 30]
f, i = torch.zeros(4), torch.zeros(4, dtype=torch.int32)
try:
    psk.psk_spmv_csr(1, 1, 1, i, i, f, f, f, ws=f)
except ValueError as e:
    assert "device tensor" in str(e)
else:
    raise AssertionError("a host tensor was taken")
print("as before")
"""


def without(prepare, words):
    r = subprocess.run([sys.executable, "-c", WITHOUT.format(prepare=prepare, words=words)], capture_output=True, text=True,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0 and "as before" in r.stdout, r.stderr


MISSING = ("sys.modules['paper_2001_00532_amd._marshal'] = None", "_marshal")
FOREIGN = ("m = types.ModuleType('paper_2001_00532_amd._marshal'); m.built_for = 'torch 1.0, Python 2.7'; sys.modules[m.__name__] = m", "torch 1.0")


@pytest.mark.parametrize("prepare,words", [MISSING, FOREIGN])
def test_everything_works_without_the_native_side(prepare, words):
    """Not built, or built for another torch: the Python functions do its work, as for tensors that are not plain."""
    without(prepare, words)


@pytest.mark.gpu
def test_products_without_the_native_side():
    without(*MISSING)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_spmv_of_plain_and_other_tensors(dtype):
    f = psk.psk_spmv_csr if dtype == torch.float32 else psk.psk_spmv_csr_f64
    op = psk.PSK_OP_SPMV_CSR if dtype == torch.float32 else psk.PSK_OP_SPMV_CSR_F64
    pos = torch.tensor([0, 2, 2, 3], dtype=torch.int32, device="cuda")
    crd = torch.tensor([0, 2, 1], dtype=torch.int32, device="cuda")
    vals = torch.tensor([1.0, 2.0, 3.0], dtype=dtype, device="cuda")
    x = torch.tensor([1.0, 10.0, 100.0], dtype=dtype, device="cuda")
    y = torch.full((3,), float("nan"), dtype=dtype, device="cuda")
    ws = psk.workspace(op, 3, 3)
    want = torch.tensor([201.0, 0.0, 30.0], dtype=dtype)
    for args in ((pos, crd, vals, x), (pos, crd, torch.nn.Parameter(vals), x), (pos, crd, vals.as_subclass(Sub), x),
                 (torch.stack([pos, pos])[1], crd, vals, torch.cat([x, x])[3:])):
        y.fill_(float("nan"))
        assert f(np.int64(3), 3, np.int32(3), *args, y, ws=ws) is y
        assert torch.equal(y.cpu(), want)
    y.fill_(float("nan"))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    f(3, 3, 3, pos, crd, vals, x, y, ws=ws, stream=s)
    s.synchronize()
    assert torch.equal(y.cpu(), want)
    with pytest.raises(ValueError, match="expected dtype"):
        f(3, 3, 3, pos.long(), crd, vals, x, y, ws=ws)
    with pytest.raises(ValueError, match="innermost"):
        f(3, 3, 3, pos, crd, vals, torch.stack([x, x], 1)[:, 0], y, ws=ws)
    with pytest.raises(psk.PskError):
        f(-1, 3, 3, pos, crd, vals, x, y, ws=ws)
    with pytest.raises(psk.PskError):
        f(3, 3, 3, pos, crd, vals, x, y, ws=ws[:16])
