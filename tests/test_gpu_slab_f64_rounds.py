"""fp64 pair sums where a chunk has about as many pairs as its staging area holds: 255, 256, 257 and 512 pairs in a chunk of 512
slots, among chunks with few.  Oracle and bar as for the other fp64 slab tests: |got - ref| <= 1e-14 * sum |a x| + 1e-300."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("pairs", [1, 255, 256, 257, 384, 511, 512])
def test_pairs_per_chunk(pairs):
    # chunks in CSR order of one slab: `pairs` rows that share 512 entries as evenly as they can
    one = np.full(pairs, 512 // pairs)
    one[:512 - one.sum()] += 1
    L = np.concatenate([one] * 3 + [[512, 1, 2, 509]] + [one] * 2 + [[77]])
    A = wl.csr_from_lengths(L, 900, seed=pairs)
    v = A.vals.astype(np.float64)
    x = wl.dense_uniform(900, 3, wl.S_B).astype(np.float64)
    S = psk.psk_slab_build_csr_f64(A.rows, 900, A.nnz, dev(A.pos), dev(A.crd), dev(v))
    y = torch.full((A.rows,), float("nan"), dtype=torch.float64, device="cuda")
    psk.psk_spmv_slab_f64(S, dev(x), y)
    torch.cuda.synchronize()
    ref, mag = oracle.spmv_csr_f64(A.pos, A.crd, v, x)
    got = y.cpu().numpy()
    assert (np.abs(got - ref) <= 1e-14 * mag + 1e-300).all(), float((np.abs(got - ref) / mag).max())
