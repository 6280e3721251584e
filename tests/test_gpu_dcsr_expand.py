"""DCSR SpMV with the row sums kept in the order of the stored rows and streamed to y in one go: the same bits as the route that
stores each row where it belongs (a workspace without room for the sums, and phases called one by one), at the edges of the
pieces in which y is written, for every alignment of y."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402

REL, FLOOR = 1e-5, 1e-30


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# rows, stored: all rows stored (in place on either workspace), one piece of 1 024, a piece and a bit, 64 and 65 entries, one row in
# sixteen (256 entries per piece) and one more, several spans, enough rows (> 16 384 pieces) that a wave writes more than one piece,
# one row in three from 2^22 rows on (six loads of entries per piece), all of 2^20 rows (kept together with three passes: 16 loads)
@pytest.mark.parametrize("passes", [1, 3])
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("rows,stored", [(1, 1), (1024, 64), (1025, 64), (1025, 65), (4099, 4099), (16_000, 1000), (16_000, 1001),
                                         (70_001, 900), (17_000_003, 5000), (4_194_304, 1_398_101), (4_194_303, 1_398_101),
                                         (1_048_576, 1_048_576)])
def test_same_bits_as_storing_rows_in_place(rows, stored, off, passes):
    rng = np.random.default_rng(rows + stored)
    L = rng.integers(0, 30, size=stored)
    L[stored // 2] = 400
    A = wl.dcsr_from_lengths(rows, L, 2011, seed=7)
    x = wl.dense_uniform(2011, 9, wl.S_X)
    args = (A.rows, A.cols, A.nnz, dev(A.crd_i), dev(A.pos), dev(A.crd), dev(A.vals), dev(x))
    full = psk.workspace(psk.PSK_OP_SPMV_CSR, A.nstored, A.nnz, tile=256)
    small = full[:full.numel() - (A.nstored * 4 + 255) // 256 * 256].clone()

    def product(ws, phases):
        y = torch.full((rows + off,), float("nan"), device="cuda")[off:]
        print("dcsr rows", rows, "stored", stored, "off", off, "passes", passes, "ws", ws.numel(), phases, flush=True)
        for ph in phases:
            psk.psk_spmv_dcsr(*args, y, tile=256, col_passes=passes, phases=ph, ws=ws)
        torch.cuda.synchronize()
        return y

    y = product(full, [psk.PSK_PHASE_ALL])
    assert torch.equal(y, product(small, [psk.PSK_PHASE_ALL]))
    assert torch.equal(y, product(full, [psk.PSK_PHASE_PARTITION, psk.PSK_PHASE_MAIN, psk.PSK_PHASE_FIXUP]))
    assert torch.equal(y, product(full, [psk.PSK_PHASE_PARTITION, psk.PSK_PHASE_MAIN | psk.PSK_PHASE_FIXUP]))
    ref, mag = oracle.spmv_dcsr(A.rows, A.crd_i, A.pos, A.crd, A.vals, x)
    ok, worst = oracle.within_tolerance(y.cpu().numpy(), ref, mag, REL, FLOOR)
    assert ok, worst


@pytest.mark.parametrize("passes", [1, 2])
@pytest.mark.parametrize("tile", [256, 2048])
def test_same_bits_around_a_long_run_of_empty_stored_rows(tile, passes):
    """A tile over more than 32 768 stored rows (empty ones are allowed) finds the rows of its positions by search on the route
    with the sums kept together and walks them on the other one: rows of less than 32 entries, of 32 and more, and the part of a
    row that an earlier tile began must be added up in the same order on both."""
    for lengths in ([100, 0], [1000, 0], [5, 31, 32, 33, 200, 0], [300, 0, 700, 0, 64, 1], [tile + 40, 0, 35]):
        L = []
        for n in lengths:
            L += [n] if n else [0] * 33_500
        L += [3] * 40 + [0, 0, 90]
        A = wl.dcsr_from_lengths(len(L) * 16 + 3, np.asarray(L), 4001, seed=len(L))
        x = wl.dense_uniform(4001, 9, wl.S_X)
        args = (A.rows, A.cols, A.nnz, dev(A.crd_i), dev(A.pos), dev(A.crd), dev(A.vals), dev(x))
        small = torch.empty(psk.psk_workspace_bytes(psk.PSK_OP_SPMV_CSR, A.nstored, A.nnz, tile=tile), dtype=torch.uint8, device="cuda")
        full = torch.empty(psk.psk_spmv_dcsr_workspace_bytes(A.nstored, A.nnz, tile), dtype=torch.uint8, device="cuda")
        got = []
        for ws, phases in ((full, [7]), (small, [7]), (full, [1, 2, 4])):
            y = torch.full((A.rows,), float("nan"), device="cuda")
            for ph in phases:
                psk.psk_spmv_dcsr(*args, y, tile=tile, col_passes=passes, phases=ph, ws=ws)
            torch.cuda.synchronize()
            got.append(y)
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2]), lengths
        ref, mag = oracle.spmv_dcsr(A.rows, A.crd_i, A.pos, A.crd, A.vals, x)
        ok, worst = oracle.within_tolerance(got[0].cpu().numpy(), ref, mag, REL, FLOOR)
        assert ok, (lengths, worst)
