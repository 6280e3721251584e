"""The native side of a call: plain tensors by their C++ object, everything else as the Python function decides."""
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
