"""SpMM tiles that sweep over the columns together and walk their rows one after the other: row ends at the first and last positions of
tiles and of the blocks that longer tiles are staged in, empty rows between, tiles with as many row ends as are still walked row by row
and with more, operands in one piece and in chunks of columns, phases one by one, NaN and Inf.  Oracle and bar as for the
other SpMM tests: |got - ref| <= 1e-5 * sum |a b| + 1e-30."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_spmm_wave import same_specials, with_specials

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def product(A, Bh, k, tile, phases=(7,)):
    C = torch.full((A.rows, k + 1), float("nan"), device="cuda")
    ws = psk.workspace(psk.PSK_OP_SPMM_CSR, A.rows, A.nnz, k=k, tile=tile)
    pos, crd, vals, B = dev(A.pos), dev(A.crd), dev(A.vals), dev(Bh)
    for ph in phases:
        psk.psk_spmm_csr(A.rows, A.cols, A.nnz, pos, crd, vals, B, C[:, :k], tile=tile, ws=ws, phases=ph)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    assert np.isnan(got[:, k:]).all(), "columns past k were written"
    return got[:, :k]


def operand(tile, k, seed):
    """From 4 300 tiles on, B of 9 MB and more, rows of several tiles in the mean."""
    rng = np.random.default_rng(seed)
    need = 4300 * tile
    runs, total = [], 0
    while total < need:
        kind = rng.integers(6)
        if kind == 0: part = [tile] * int(rng.integers(1, 4))                        # ends at the last position of a tile
        elif kind == 1: part = [2 * tile - 1, 1, 2 * tile + 1, tile - 1]             # ... at the first, the last but one
        elif kind == 2: part = [0, 0, 3 * tile // 2, 0, 5, 1, 0, 2 * tile]           # few ends in a tile, empty rows
        elif kind == 3: part = list(rng.integers(0, 6, size=10)) + [4 * tile]        # many
        elif kind == 4: part = [576, 577, 575, 1152]                                 # ends at blocks of long tiles
        else: part = [int(rng.integers(8 * tile, 12 * tile))] * 12
        runs += part
        total += sum(part)
    cols = max((9 << 20) // (4 * k) + 7, 12 * tile)
    A = wl.csr_from_lengths(np.array(runs), cols, seed=seed)
    assert A.rows * tile <= 0.8 * A.nnz and 2 * cols * A.rows <= 768 * A.nnz
    return A, wl.dense_uniform(cols * k, 3, wl.S_B).reshape(cols, k)


@pytest.mark.parametrize("tile,k", [(256, 20), (256, 33), (256, 64), (256, 100), (256, 128), (256, 260), (512, 16), (512, 32), (1024, 24), (1024, 96)])
def test_row_ends(tile, k):
    A, Bh = operand(tile, k, tile + k)
    ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
    got = product(A, Bh, k, tile)
    ok, worst = oracle.within_tolerance(got, ref, mag)
    assert ok, "%.3g of the bar" % worst
    assert (product(A, Bh, k, tile, (1, 2, 4)) == got).all(), "one phase at a time"


@pytest.mark.parametrize("tile,k", [(256, 32), (256, 64), (512, 24), (1024, 96)])
def test_nan_inf_and_overflow_reach_only_their_rows(tile, k):
    """In short rows of tiles with more row ends than are walked row by row, and in rows of several tiles."""
    A, Bh = operand(tile, k, 5)
    lengths = np.diff(A.pos)
    first = A.pos[:-1] // tile
    ends = np.bincount(A.pos[1:][lengths > 0] // tile, minlength=A.nnz // tile + 2)          # about: rows that end in each tile
    short, long = (lengths >= 3) & (lengths < 8) & (ends[first] > 5), lengths > 2 * tile
    rows = np.sort(np.concatenate([np.flatnonzero(short)[::2], np.flatnonzero(long)[::3]]))
    A, count = with_specials(A, np.random.default_rng(k), rows=rows)
    assert short.sum() >= 100 and long.sum() >= 100 and (count >= 10).all()
    Bh[0], Bh[1], Bh[2], Bh[3] = np.nan, np.inf, -np.inf, 2e38
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
    same_specials(product(A, Bh, k, tile), ref, mag)
