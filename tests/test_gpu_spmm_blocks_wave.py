"""Block SpMM of up to 64 columns, a wave per tile: group widths, block rows that end inside a group's run, at its borders and
behind the tile, empty block rows (more than 16 bits number among them), few and many tiles, NaN and Inf.  Oracle and bar as for
the other SpMM tests: |got - ref| <= 1e-5 * sum |a b| + 1e-30."""
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


def product(A, bs, Bh, k, tile=0, phases=(7,)):
    C = torch.full((A.rows * bs, k + 1), float("nan"), device="cuda")
    ws = psk.workspace(psk.PSK_OP_SPMM_BCSR, A.rows, A.nnz, k=k, bs=bs, tile=tile)
    pos, crd, vals, B = dev(A.pos), dev(A.crd), dev(A.vals), dev(Bh)[:, :k]
    for ph in phases:
        psk.psk_spmm_bcsr(A.rows, A.cols, A.nnz, bs, pos, crd, vals, B, C[:, :k], tile=tile, ws=ws, phases=ph)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    assert np.isnan(got[:, k:]).all(), "columns past k were written"
    return got[:, :k]


PATTERNS = {"short": [0, 1, 2, 3, 9], "middle": [5, 8, 12], "long": [0, 1, 63, 64, 65, 96, 97, 200, 290]}


@pytest.mark.parametrize("bs", [2, 4, 8])
@pytest.mark.parametrize("k", [4, 5, 8, 9, 16, 17, 32, 33, 48, 64])
def test_widths(bs, k):
    for pattern, lengths in PATTERNS.items():
        rng = np.random.default_rng(k + bs)
        L = rng.choice(lengths, size=41_000 // int(np.mean(lengths)) + 400)
        A = wl.csr_from_lengths(L, 300, seed=k, bs=bs)
        assert A.nnz >= 600 * 64
        Bh = wl.dense_uniform(300 * bs * (k + 1), 3, wl.S_B).reshape(300 * bs, k + 1)
        ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, np.ascontiguousarray(Bh[:, :k]), bs)
        got = product(A, bs, Bh, k)
        ok, worst = oracle.within_tolerance(got, ref, mag)
        assert ok, "bs %d k %d %s: %.3g of the bar" % (bs, k, pattern, worst)
        assert (product(A, bs, Bh, k, 0, (1, 2, 4)) == got).all(), "one phase at a time"


@pytest.mark.parametrize("bs,k,rows,tile", [(4, 8, 1, 0), (8, 32, 3, 0), (4, 20, 40, 512), (8, 4, 200, 256)])
def test_few_tiles(bs, k, rows, tile):
    A = wl.csr_from_lengths(np.full(rows, 37), 300, seed=k, bs=bs)
    Bh = wl.dense_uniform(300 * bs * (k + 1), 3, wl.S_B).reshape(300 * bs, k + 1)
    ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, np.ascontiguousarray(Bh[:, :k]), bs)
    ok, worst = oracle.within_tolerance(product(A, bs, Bh, k, tile), ref, mag)
    assert ok, "%.3g of the bar" % worst


def test_runs_of_empty_block_rows():
    L = np.concatenate([[3, 0, 5], np.zeros(70_000, dtype=int), [2, 7], np.zeros(500, dtype=int), [9] * 30])
    A = wl.csr_from_lengths(L, 300, seed=2, bs=4)
    Bh = wl.dense_uniform(300 * 4 * 13, 3, wl.S_B).reshape(1200, 13)
    ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, np.ascontiguousarray(Bh[:, :12]), 4)
    ok, worst = oracle.within_tolerance(product(A, 4, Bh, 12), ref, mag)
    assert ok, "%.3g of the bar" % worst


@pytest.mark.parametrize("length", [3, 9, 70])
@pytest.mark.parametrize("bs,k", [(2, 24), (2, 7), (4, 8), (4, 32), (4, 48), (8, 16), (8, 64)])
def test_nan_inf_and_overflow_reach_only_their_block_rows(bs, k, length):
    """Block column 0 among them: places that hold no block must not bring it in.  (8 x 8: the same kinds in the first column of the block.)"""
    rng = np.random.default_rng(bs + length)
    A = wl.csr_from_lengths(np.full(600 * 64 // length + 40, length), 300, seed=bs, bs=bs)
    assert A.nnz >= 600 * 64
    A, count = with_specials(A, rng, bs)
    assert (count >= 10).all()
    Bh = wl.dense_uniform(300 * bs * k, 3, wl.S_B).reshape(300 * bs, k)
    Bh[0], Bh[bs], Bh[2 * bs], Bh[3 * bs] = np.nan, np.inf, -np.inf, 2e38
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, Bh, bs)
    same_specials(product(A, bs, Bh, k), ref, mag)


@pytest.mark.parametrize("bs,k", [(2, 8), (2, 40), (4, 5), (4, 32), (4, 64), (8, 12), (8, 48)])
def test_offsets_beyond_32_bits(bs, k):
    """B as rows far apart: from 2^30 floats of rows * ldb on the byte offsets into B don't fit 32 bits.  One row stride on either side, the last
    rows of B referred to."""
    cols = 280
    A = wl.csr_from_lengths(np.full(5500, 8), cols, seed=k, bs=bs)
    assert A.crd.max() == cols - 1 and A.nnz >= 600 * 64
    n = cols * bs
    Bh = wl.dense_uniform(n * k, 5, wl.S_B).reshape(n, k)
    ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, Bh, bs)
    most = (2 ** 32 - 1) // 4 // n
    buf = torch.empty(n * (most + 1), device="cuda")
    for ld in (most, most + 1):
        B = buf[:n * ld].view(n, ld)[:, ld - k:]
        B.copy_(dev(Bh))
        C = torch.full((A.rows * bs, k), float("nan"), device="cuda")
        print("bcsr spmm wave offsets bs", bs, "k", k, "ld", ld, flush=True)
        psk.psk_spmm_bcsr(A.rows, cols, A.nnz, bs, dev(A.pos), dev(A.crd), dev(A.vals), B, C)
        torch.cuda.synchronize()
        ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, mag)
        assert ok, "bs %d k %d ld %d: %.3g of the bar" % (bs, k, ld, worst)


@pytest.mark.parametrize("bs,k,pad,per,brows", [(2, 12, 0, 1, 60_000), (2, 17, 3, 1, 60_000), (4, 25, 0, 1, 50_000), (4, 61, 1, 2, 30_000), (8, 57, 0, 1, 40_000), (8, 5, 2, 3, 20_000),
                                                (2, 45, 0, 1, 570_000), (4, 9, 0, 0, 1_450_000), (4, 61, 0, 2, 210_000), (8, 45, 0, 1, 145_000), (4, 48, 0, 1, 270_000),
                                                (4, 20, 0, 2, 16), (4, 20, 0, 2, 17), (8, 9, 1, 2, 8), (8, 9, 1, 2, 9), (2, 30, 0, 3, 30_000)])
def test_few_blocks_per_row(bs, k, pad, per, brows):
    """Rows of C that share 64-byte pieces with their neighbours, C below and above the size up to which they go through the L2, and the
    products that go to the workgroups' kernel.  per = 0: one block row in four has a block."""
    rng = np.random.default_rng(k)
    A = wl.csr_from_lengths(np.full(brows, per) if per else (rng.random(brows) < 0.25).astype(np.int64), 300, seed=k, bs=bs)
    Bh = wl.dense_uniform(300 * bs * k, 3, wl.S_B).reshape(300 * bs, k)
    C = torch.full((A.rows * bs, k + pad), float("nan"), device="cuda")
    psk.psk_spmm_bcsr(A.rows, 300, A.nnz, bs, dev(A.pos), dev(A.crd), dev(A.vals), dev(Bh), C[:, :k])
    got = C.cpu().numpy()
    assert np.isnan(got[:, k:]).all(), "columns past k were written"
    ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, Bh, bs)
    ok, worst = oracle.within_tolerance(got[:, :k], ref, mag)
    assert ok, "%.3g of the bar" % worst


@pytest.mark.parametrize("bs,k,full", [(4, 28, 32), (2, 45, 48)])
def test_narrow_rows_take_no_longer_than_wide_ones(bs, k, full):
    """300 000 rows of one block: stored past the L2 one by one, rows that share 64-byte pieces of C took 1.7 times as long as wider ones that
    fill them (4 x 4 66.6 us against 38.3, now 40.9)."""
    A = wl.csr_from_lengths(np.ones(300_000 if bs == 4 else 400_000, dtype=np.int64), 4000, seed=1, bs=bs)
    pos, crd, vals = dev(A.pos), dev(A.crd), dev(A.vals)
    ws = psk.workspace(psk.PSK_OP_SPMM_BCSR, A.rows, A.nnz, k=full, bs=bs)
    took = {}
    for n in (k, full):
        B = dev(wl.dense_uniform(4000 * bs * n, 3, wl.S_B).reshape(4000 * bs, n))
        C = torch.empty((A.rows * bs, n), device="cuda")
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                psk.psk_spmm_bcsr(A.rows, 4000, A.nnz, bs, pos, crd, vals, B, C, ws=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[n] = min(times)
    print(took, flush=True)
    assert took[k] <= 1.35 * took[full]
