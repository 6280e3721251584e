"""SpMM where its kernels change over and where tiles hand rows to each other: numbers of columns around the group widths,
rows that reach a little (finished by the tile they begin in) or far (carried) past a tile's end, rows of one and two entries
(several ends in one step), operands whose rows are not aligned.  Oracle and bar as for the other SpMM tests:
|got - ref| <= 1e-5 * sum |a b| + 1e-30 per element."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(lengths, k, tile, bs=1, pad=1):
    cols = 900
    A = wl.csr_from_lengths(np.asarray(lengths), cols, seed=k + 1, bs=bs)
    Bh = wl.dense_uniform(cols * bs * (k + pad), 3, wl.S_B).reshape(cols * bs, k + pad)
    Bd = dev(Bh)[:, :k]
    C = torch.full((A.rows * bs, k + pad), float("nan"), device="cuda")
    if bs == 1:
        psk.psk_spmm_csr(A.rows, cols, A.nnz, dev(A.pos), dev(A.crd), dev(A.vals), Bd, C[:, :k], tile=tile)
        ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh[:, :k])
    else:
        psk.psk_spmm_bcsr(A.rows, cols, A.nnz, bs, dev(A.pos), dev(A.crd), dev(A.vals), Bd, C[:, :k], tile=tile)
        ref, mag = oracle.spmm_bcsr(A.pos, A.crd, A.vals, np.ascontiguousarray(Bh[:, :k]), bs)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    assert np.isnan(got[:, k:]).all(), "columns past k were written"
    ok, worst = oracle.within_tolerance(got[:, :k], ref, mag)
    assert ok, "k %d tile %d bs %d: %.3g of the bar" % (k, tile, bs, worst)


def borders(T):
    """Rows that end 1 before, at, and 1 behind a tile's end, at the last position still taken over, one behind it, two tiles on;
    short rows behind them keep the mean below the length from which nothing is taken over."""
    return long_borders(T) + [1] * 50


def long_borders(T):
    h = T // 2
    return [T - 1, 2, T - 1 + h, 0, 0, T - h, h + 1 + T, 1, 1, T - 3 - h, 3 * T + h, 2 * T - 1, 5, 0, T]


@pytest.mark.parametrize("k", [1, 3, 4, 5, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 67, 99, 127, 128, 129])
def test_group_widths_and_tile_borders(k):
    check(borders(256), k, 256)
    check(long_borders(256), k, 256)
    rng = np.random.default_rng(k)
    check(rng.choice([0, 1, 2, 3, 9], size=1500), k, 0, pad=0)           # several row ends in one step
    check(np.full(300, 40), k, 512, pad=4)


@pytest.mark.parametrize("bs,k", [(2, 33), (4, 64), (4, 130), (8, 20)])
def test_block_rows_at_tile_borders(bs, k):
    check(borders(64), k, 64, bs=bs)
    check([133, 300, 0, 64, 400, 0, 500, 192, 1], k, 64, bs=bs)          # (a mean of two tiles and more: no tails)
    check(np.full(200, 8), k, 0, bs=bs, pad=0)


@pytest.mark.parametrize("k,tile,cols,per_row", [(32, 0, 70_000, 2200), (48, 256, 50_000, 1300), (128, 0, 30_000, 2200),
                                                 (31, 512, 90_000, 4000)])
def test_tiles_in_column_order(k, tile, cols, per_row):
    """Long rows and a B of 8 MB and more: the tiles are worked on by the column they begin with.  Sorted and unsorted columns,
    rows of very different lengths among them, empty rows at both ends."""
    rows = 4200 * 512 // per_row if tile != 256 else 4200 * 256 // per_row
    rng = np.random.default_rng(k)
    L = np.full(rows, per_row)
    L[rng.integers(0, rows, 20)] = rng.integers(0, 3 * per_row, 20)
    L[[0, rows - 1]] = 0
    L[1] += max(0, 4096 * (tile or 512) + 1 - int(L.sum()))
    assert L.max() <= cols
    A = wl.csr_from_lengths(L, cols, seed=k)
    crd = A.crd.copy()
    half = A.nnz // 2
    crd[half:] = rng.integers(0, cols, A.nnz - half)                      # the second half: any order, repeated columns
    Bh = wl.dense_uniform(cols * k, 4, wl.S_B).reshape(cols, k)
    C = torch.full((rows, k), float("nan"), device="cuda")
    psk.psk_spmm_csr(rows, cols, A.nnz, dev(A.pos), dev(crd), dev(A.vals), dev(Bh), C, tile=tile)
    torch.cuda.synchronize()
    ref, mag = oracle.spmm_csr(A.pos, crd, A.vals, Bh)
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, mag)
    assert ok, "k %d tile %d: %.3g of the bar" % (k, tile, worst)


def wave_shares(pos, crd, vals, B, share, bs):
    """Rows summed in fp32, one product after the other (fused multiply-adds) inside shares of `share` positions, and the
    shares of a row in fp64: a tile of 4 * share positions cut among its four waves."""
    per = int(pos[1])
    rows, k = pos.size - 1, B.shape[1]
    v = vals.reshape(rows, per, bs, bs).astype(np.float64)
    b = B.reshape(-1, bs, k)[crd].reshape(rows, per, bs, k).astype(np.float64)
    out = np.zeros((rows, bs, k))
    acc = np.zeros((rows, bs, k), dtype=np.float32)
    for i in range(per):
        new = (pos[:-1] + i) % share == 0
        out[new] += acc[new]
        acc[new] = 0
        for j in range(bs):
            acc = (acc + v[:, i, :, j, None] * b[:, i, j, None, :]).astype(np.float32)
    return (out + acc).reshape(rows * bs, k)


@pytest.mark.parametrize("rows,per,k,bs", [(4000, 300, 128, 1), (6000, 70, 200, 1), (3000, 640, 128, 1), (20_000, 8, 64, 4), (8000, 20, 130, 2),
                                           (4000, 6, 64, 8)])
def test_error_is_not_above_that_of_the_cut(rows, per, k, bs):
    """The error of the sums (positive operands: rounding is all there is) against that of the cut as it stands, tiles of the
    default size with a quarter for each wave and fp64 across: a row tail that its tile finishes must not make it larger.
    (rms over 10^5 elements and more: the two differ by chance by less than 1 %; 5 % is allowed.)"""
    cols = 3000
    rng = np.random.default_rng(per)
    A = wl.csr_from_lengths(np.full(rows, per), cols, seed=per, bs=bs)
    vals = rng.random(A.vals.size, dtype=np.float32)
    B = rng.random((cols * bs, k), dtype=np.float32)
    C = torch.empty((rows * bs, k), device="cuda")
    if bs == 1:
        psk.psk_spmm_csr(rows, cols, A.nnz, dev(A.pos), dev(A.crd), dev(vals), dev(B), C)
    else:
        psk.psk_spmm_bcsr(rows, cols, A.nnz, bs, dev(A.pos), dev(A.crd), dev(vals), dev(B), C)
    few = slice(0, 24)                                     # (columns are summed alike)
    share = psk.psk_default_tile(psk.PSK_OP_SPMM_CSR if bs == 1 else psk.PSK_OP_SPMM_BCSR) // 4
    v = vals.reshape(rows, per, bs, bs).astype(np.float64)
    b = B[:, few].reshape(cols, bs, -1).astype(np.float64)[A.crd].reshape(rows, per, bs, -1)
    exact = np.einsum("rpij,rpjk->rik", v, b).reshape(rows * bs, -1)
    rms = lambda got: float(np.sqrt(np.mean(((got - exact) / exact) ** 2)))
    here, cut = rms(C[:, few].cpu().numpy()), rms(wave_shares(A.pos, A.crd, vals, B[:, few], share, bs))
    print("spmm error", rows, per, k, bs, here, cut, flush=True)
    assert here <= 1.05 * cut


@pytest.mark.parametrize("k", [1, 3, 4, 8, 16, 32, 64])
def test_waves_parts_of_a_row_are_added_in_fp64(k):
    """Group kernels, one row over a tile: 2^24 in the first wave's share, a 1 in each of two others.  Added to 2^24 in fp32 one
    after the other both would be lost; in fp64 they count (2^24 + 2 is a float)."""
    vals = np.zeros(512, dtype=np.float32)
    vals[[0, 200, 400]] = 2.0 ** 24, 1.0, 1.0
    B, C = torch.ones((1, k), device="cuda"), torch.empty((1, k), device="cuda")
    psk.psk_spmm_csr(1, 1, 512, dev(np.array([0, 512], dtype=np.int32)), torch.zeros(512, dtype=torch.int32, device="cuda"), dev(vals), B, C,
                     tile=512)
    assert bool((C == 2.0 ** 24 + 2).all())


@pytest.mark.parametrize("k", [3, 8, 16, 32, 64, 99])
def test_offsets_beyond_32_bits(k):
    """B as rows far apart: from 2^30 floats of cols * ldb on the byte offsets into B don't fit 32 bits (another instance of the
    group kernels).  One row stride on either side, the last rows of B referred to."""
    cols, per = 1100, 60
    A = wl.csr_from_lengths(np.full(300, per), cols, seed=k)
    assert A.crd.max() == cols - 1
    Bh = wl.dense_uniform(cols * k, 5, wl.S_B).reshape(cols, k)
    ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
    most = (2 ** 32 - 1) // 4 // cols
    buf = torch.empty(cols * (most + 1), device="cuda")
    for ld in (most, most + 1):
        B = buf[:cols * ld].view(cols, ld)[:, ld - k:]            # the last columns: offsets up to the end of the buffer
        B.copy_(dev(Bh))
        C = torch.full((300, k), float("nan"), device="cuda")
        print("spmm offsets k", k, "ld", ld, flush=True)
        psk.psk_spmm_csr(300, cols, A.nnz, dev(A.pos), dev(A.crd), dev(A.vals), B, C)
        torch.cuda.synchronize()
        ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, mag)
        assert ok, "k %d ld %d: %.3g of the bar" % (k, ld, worst)
