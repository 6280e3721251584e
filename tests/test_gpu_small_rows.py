"""Small products: blocks of whole rows in one launch (around the lengths at which a row is summed by a thread, a wave, a
workgroup, around chunks, blocks and the size limits), the tile kernels that search their rows themselves (few tiles), and
the clearing of long runs of empty rows, which the fix-up step finds from the table.  Bars: |got - ref| <= 1e-5 (fp64: 1e-14)
* sum |a x| + 1e-30 (1e-300) per row; every row of y is preset to NaN."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(lengths, f64, tile=0, cols=70_000, phases=(7,), seed=1):
    A = wl.csr_from_lengths(np.asarray(lengths, dtype=np.int64), cols, seed=seed)
    pos, crd = dev(A.pos), dev(A.crd)
    if f64:
        v, x = wl.dense_uniform_f64(A.nnz, 3, wl.S_VALS), wl.dense_uniform_f64(cols, 3, wl.S_X)
        ref, mag = oracle.spmv_csr_f64(A.pos, A.crd, v, x)
        f, op, bar = psk.psk_spmv_csr_f64, psk.PSK_OP_SPMV_CSR_F64, (1e-14, 1e-300)
    else:
        v, x = A.vals, wl.dense_uniform(cols, 3, wl.S_X)
        ref, mag = oracle.spmv_csr(A.pos, A.crd, v, x)
        f, op, bar = psk.psk_spmv_csr, psk.PSK_OP_SPMV_CSR, (1e-5, 1e-30)
    y = torch.full((A.rows,), float("nan"), dtype=torch.float64 if f64 else torch.float32, device="cuda")
    ws = psk.workspace(op, A.rows, A.nnz, tile=tile)
    ws.fill_(0x7f)
    for p in phases:
        f(A.rows, cols, A.nnz, pos, crd, dev(v), dev(x), y, tile=tile, phases=p, ws=ws)
    torch.cuda.synchronize()
    ok, worst = oracle.within_tolerance(y.cpu().numpy(), ref, mag, *bar)
    assert ok, "worst |err|/bar = %.3g" % worst


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("lengths", [
    [31, 32, 33, 0, 511, 512, 513, 1], [8191], [8192], [8193], [8192 - 600, 600, 600], [0, 0, 24576], [24577], [5] * 1023,
    [5] * 1024, [5] * 1025, [1] * 4096, [0] * 65535 + [7], [0] * 65536 + [7], [9000, 0, 9000, 3], [512] * 16 + [32] * 256,
], ids=lambda v: "%dx%d" % (len(v), max(v)))
def test_row_blocks(lengths, f64):
    check(lengths, f64)


@pytest.mark.parametrize("n", [49151, 49152, 49153])
def test_size_limit_of_the_one_launch_path(n):
    check([n], False)
    check([n // 3, n - n // 3 - 7, 7], False)


@pytest.mark.parametrize("f64,n,tiles", [(False, 24576, False), (False, 24577, True), (False, 49152, True),
                                         (True, 12288, False), (True, 12289, True), (True, 24576, True)])
def test_one_long_row_goes_by_tiles(f64, n, tiles):
    """A row is one workgroup's in the row blocks; by tiles its later parts wait for the fix-up step.  (All terms are 1.)"""
    dt, tile = (torch.float64, 1024) if f64 else (torch.float32, 2048)
    f, op = (psk.psk_spmv_csr_f64, psk.PSK_OP_SPMV_CSR_F64) if f64 else (psk.psk_spmv_csr, psk.PSK_OP_SPMV_CSR)
    check([n], f64)
    check([n], f64, phases=(1, 2, 4))
    pos = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    crd = torch.arange(n, dtype=torch.int32, device="cuda") % 3000
    ws = psk.workspace(op, 1, n)
    y = torch.full((1,), float("nan"), dtype=dt, device="cuda")
    args = (1, 3000, n, pos, crd, torch.ones(n, dtype=dt, device="cuda"), torch.ones(3000, dtype=dt, device="cuda"), y)
    f(*args, phases=psk.PSK_PHASE_PARTITION | psk.PSK_PHASE_MAIN, ws=ws)
    assert y.item() == (tile if tiles else n)
    f(*args, phases=psk.PSK_PHASE_FIXUP, ws=ws)
    assert y.item() == n


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("tile", [256, 1024])
@pytest.mark.parametrize("phases", [(7,), (1, 2, 4), (7, 6)], ids=str)
def test_tiles_that_search_their_rows(tile, phases, f64):
    rng = np.random.default_rng(tile)
    check(rng.choice([0, 1, 3, 20, 700], size=3000, p=[.3, .3, .2, .19, .01]), f64, tile, phases=phases)
    check([tile] * 5 + [tile // 2] * 3, f64, tile, phases=phases)
    check([3 * tile + 5, 0, 2], f64, tile, phases=phases)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rows", [32768, 32769, 40961, 100_000, 8192 * 13, 8192 * 13 + 1])
def test_long_runs_of_empty_rows_without_a_list(rows, f64):
    for filled in ([0], [rows - 1], [rows // 2], [0, rows - 1], [8191, 8192, 8193, 40_000 % rows], [5, 33_000 % rows, rows - 2]):
        L = np.zeros(rows, dtype=np.int64)
        for i, r in enumerate(filled):
            L[r] = (3, 700, 256, 1)[i % 4]
        check(L, f64, 256)
        check(L, f64, 1024, phases=(1, 2, 4))


@pytest.mark.parametrize("f64,lengths", [(False, [3] * 7000), (False, [0, 0, 20_000, 5, 0, 9000, 0]), (False, [0] * 40_000 + [300] * 60 + [0]),
                                         (True, [3] * 800), (True, [0, 5000, 0, 1]), (True, [0] * 40_000 + [300] * 60)],
                         ids=lambda v: "%dx%d" % (len(v), max(v)) if isinstance(v, list) else "f64" if v else "f32")
def test_phases_of_a_small_product_with_other_calls(f64, lengths):
    """The phases of a small product leave what a larger one's do: the table serves calls that give the tile's size (and, in
    fp32, entry points that share it), and a fix-up with the default tile finishes a main phase with the size given.  The
    workspace starts out as rows that exist, so that a word that was not written cannot send a kernel out of bounds."""
    A = wl.csr_from_lengths(np.asarray(lengths, dtype=np.int64), 30_000, seed=2)
    tile = 1024 if f64 else 2048
    if f64:
        v, x = wl.dense_uniform_f64(A.nnz, 3, wl.S_VALS), wl.dense_uniform_f64(30_000, 3, wl.S_X)
        (ref, mag), f, op, bar = oracle.spmv_csr_f64(A.pos, A.crd, v, x), psk.psk_spmv_csr_f64, psk.PSK_OP_SPMV_CSR_F64, (1e-14, 1e-300)
    else:
        v, x = A.vals, wl.dense_uniform(30_000, 3, wl.S_X)
        (ref, mag), f, op, bar = oracle.spmv_csr(A.pos, A.crd, v, x), psk.psk_spmv_csr, psk.PSK_OP_SPMV_CSR, (1e-5, 1e-30)
    pos = dev(A.pos)
    args = (A.rows, 30_000, A.nnz, pos, dev(A.crd), dev(v), dev(x))
    table = psk.psk_partition_csr(pos, A.nnz, tile)
    part, main, fix = psk.PSK_PHASE_PARTITION, psk.PSK_PHASE_MAIN, psk.PSK_PHASE_FIXUP
    orders = [[(f, 0, part), (f, tile, main | fix)], [(f, 0, 7), (f, tile, main), (f, tile, fix)], [(f, 0, main), (f, 0, fix)],
              [(f, tile, part | main), (f, 0, fix)], [(f, 0, main | fix), (f, 0, fix)], [(f, 0, part), (f, 0, main), (f, 0, fix)]]
    if not f64:
        orders += [[(f, 0, part), (g, 0, main | fix)] for g in (psk.psk_spmv_csr_notemp, psk.psk_spmv_csr_atomics)]
    for calls in orders:
        ws = psk.workspace(op, A.rows, A.nnz)
        ws.zero_()
        y = torch.full((A.rows,), float("nan"), dtype=torch.float64 if f64 else torch.float32, device="cuda")
        for g, t, phases in calls:
            print("small phases", g.__name__, "tile", t, "phases", phases, "nnz", A.nnz, flush=True)
            g(*args, y, tile=t, phases=phases, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(ws[:table.numel() * 4].view(torch.int32), table)
        ok, worst = oracle.within_tolerance(y.cpu().numpy(), ref, mag, *bar)
        assert ok, (calls, worst)


@pytest.mark.parametrize("n", [20_000, 49_152])
def test_parts_of_a_long_row_are_added_in_fp64(n):
    """A product 2^24, four products 1 further on, zeros in between: in fp32 every 1 would be lost against 2^24, added up among
    themselves and in fp64 they count.  (Four 1s: the sum is a float.)"""
    vals = np.zeros(n, dtype=np.float32)
    vals[0] = 2.0 ** 24
    ones = np.arange(2500, n, 4500)[:4]                    # in other tiles of 2048, held by other waves, two in other chunks
    vals[ones] = 1.0
    y = torch.empty(1, device="cuda")
    one = torch.ones(1, device="cuda")
    psk.psk_spmv_csr(1, 1, n, dev(np.array([0, n], dtype=np.int32)), torch.zeros(n, dtype=torch.int32, device="cuda"), dev(vals), one, y)
    assert float(y) == 2.0 ** 24 + len(ones)
