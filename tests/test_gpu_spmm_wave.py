"""SpMM with many tiles, where a wave works on a tile alone (1536 tiles and more): group widths, rows that end inside a group's
run, at its borders and behind the tile, blocks without a row end, tiles staged in several blocks, runs of more empty rows
than 16 bits number, NaN and Inf.  Oracle and bar as for the other SpMM tests: |got - ref| <= 1e-5 * sum |a b| + 1e-30."""
import dataclasses

import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402

NNZ = 1536 * 256 + 77                        # many tiles of 256, the last one short


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rows_of(pattern, rng, nnz):
    if pattern == "short":
        L = rng.choice([0, 1, 2, 3, 9], size=nnz)
    elif pattern == "middle":
        L = rng.integers(10, 60, size=nnz // 10)
    else:
        L = rng.choice([0, 1, 255, 256, 257, 384, 385, 700, 890], size=nnz // 200)
    return L[:int(np.searchsorted(np.cumsum(L), nnz))]


def product(A, cols, Bh, k, tile, phases=(7,), pad=1):
    Bd = dev(Bh)[:, :k]
    C = torch.full((A.rows, k + pad), float("nan"), device="cuda")
    ws = psk.workspace(psk.PSK_OP_SPMM_CSR, A.rows, A.nnz, k=k, tile=tile)
    for ph in phases:
        psk.psk_spmm_csr(A.rows, cols, A.nnz, dev(A.pos), dev(A.crd), dev(A.vals), Bd, C[:, :k], tile=tile, ws=ws, phases=ph)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    assert np.isnan(got[:, k:]).all(), "columns past k were written"
    return got[:, :k]


@pytest.mark.parametrize("pattern", ["short", "middle", "long"])
@pytest.mark.parametrize("k", [4, 5, 8, 9, 16, 31, 32, 33, 64, 67, 128, 131, 256, 260])
def test_group_widths(k, pattern):
    rng = np.random.default_rng(k)
    for tile, nnz in ((256, NNZ), (2048, 1536 * 2048 + 5)) if k in (8, 33) else ((256, NNZ),):
        A = wl.csr_from_lengths(rows_of(pattern, rng, nnz + 1000), 900, seed=k)
        assert A.nnz >= 1536 * tile
        Bh = wl.dense_uniform(900 * (k + 1), 3, wl.S_B).reshape(900, k + 1)
        ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh[:, :k])
        got = product(A, 900, Bh, k, tile)
        ok, worst = oracle.within_tolerance(got, ref, mag)
        assert ok, "k %d tile %d %s: %.3g of the bar" % (k, tile, pattern, worst)
        assert (product(A, 900, Bh, k, tile, (1, 2, 4)) == got).all(), "one phase at a time"


def test_runs_of_empty_rows():
    rng = np.random.default_rng(1)
    part = rng.choice([1, 2, 40], size=10_000)
    L = np.concatenate([part, np.zeros(150_000, dtype=part.dtype), part, np.zeros(66_000, dtype=part.dtype), part, part])
    A = wl.csr_from_lengths(L, 900, seed=1)
    assert A.nnz >= 1536 * 256
    Bh = wl.dense_uniform(900 * 18, 3, wl.S_B).reshape(900, 18)
    ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh[:, :17])
    ok, worst = oracle.within_tolerance(product(A, 900, Bh, 17, 256), ref, mag)
    assert ok, "%.3g of the bar" % worst


def with_specials(A, rng, bs=1, rows=None):
    """Every 7th row of three entries and more (or every one of `rows`) refers to NaN, to Inf, to -Inf, to both, or to three finite products
    whose sum passes the fp32 range (rows 0 to 3 of B; of blocks their first rows), at early, middle and last places of the row;
    nobody else does.  The number of entries of each kind."""
    crd, vals = np.maximum(A.crd, 4), A.vals.reshape(A.nnz, bs, bs).copy()
    lengths = np.diff(A.pos)
    count = np.zeros(4, dtype=int)
    for i, r in enumerate(np.flatnonzero(lengths >= 3)[::7] if rows is None else rows):
        n = int(lengths[r])
        at = [int(rng.integers(min(n, 8))), int(rng.integers(n)), n - 1][(i // 5) % 3]
        kinds = ((0,), (1,), (2,), (1, 2), (3, 3, 3))[i % 5]
        for m, c in enumerate(kinds):
            p = A.pos[r] + (at + m) % n
            crd[p], vals[p, :, 0] = c, 1.0
            count[c] += 1
    return dataclasses.replace(A, crd=crd, vals=vals.reshape(A.vals.shape)), count


def same_specials(got, ref, mag):
    """As the sum in 64 bits, rounded: NaN, infinities (an overflow among them) and the rest within the bar."""
    with np.errstate(over="ignore", invalid="ignore"):
        want = ref.astype(np.float32)
        assert np.isnan(want).any() and np.isposinf(want).any() and np.isneginf(want).any() and (np.isinf(want) & np.isfinite(ref)).any()
        assert (np.isnan(got) == np.isnan(want)).all(), "%d places are NaN and should not be" % (np.isnan(got) & ~np.isnan(want)).sum()
        inf = np.isinf(want)
        assert (np.isinf(got) == inf).all() and (got[inf] == want[inf]).all()
        fin = np.isfinite(want)
        assert (np.abs(got[fin] - ref[fin]) <= 1e-5 * mag[fin] + 1e-30).all()


@pytest.mark.parametrize("length", [5, 16, 100, 700])
@pytest.mark.parametrize("k,tile", [(7, 256), (32, 256), (128, 256), (200, 256), (32, 2048)])
def test_nan_inf_and_overflow_reach_only_their_rows(k, tile, length):
    """Row 0 of B among them: places of a block that hold no entry must not bring it in."""
    rng = np.random.default_rng(k + length)
    tiles = 6000 if k <= 8 else 1536
    A = wl.csr_from_lengths(np.full((tiles * tile + 77) // length + 2, length), 900, seed=k)
    assert A.nnz >= tiles * tile
    A, count = with_specials(A, rng)
    assert (count >= 10).all()
    Bh = wl.dense_uniform(900 * (k + 1), 3, wl.S_B).reshape(900, k + 1)
    Bh[0], Bh[1], Bh[2], Bh[3] = np.nan, np.inf, -np.inf, 2e38
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh[:, :k])
    same_specials(product(A, 900, Bh, k, tile), ref, mag)


@pytest.mark.parametrize("k,cols,pattern", [(64, 22_000, "short"), (96, 15_000, "middle"), (128, 12_000, "long"), (128, 30_000, "short"),
                                            (256, 9_000, "middle"), (320, 12_000, "short")])
def test_columns_in_chunks(k, cols, pattern):
    """Rows of B that begin 128-byte lines and a B above the L2's size; long and short rows."""
    rng = np.random.default_rng(k)
    A = wl.csr_from_lengths(rows_of(pattern, rng, NNZ + 1000), cols, seed=k)
    Bh = wl.dense_uniform(cols * k, 3, wl.S_B).reshape(cols, k)
    ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
    for pad in (1, 32):                      # rows of C that share 64-byte pieces with their neighbours, and that fill them
        ok, worst = oracle.within_tolerance(product(A, cols, Bh, k, 256, pad=pad), ref, mag)
        assert ok, "%.3g of the bar" % worst


@pytest.mark.parametrize("k", [4, 7, 8, 12, 16, 24, 32, 40, 64, 100, 128, 160, 256])
def test_few_entries_per_row(k):
    """Rows of none to three entries, whose stores are most of the product: rows of C that share 64-byte pieces (stored through the
    L2 or by a workgroup) and that fill them; rows that are mostly empty."""
    rng = np.random.default_rng(k)
    patterns = ((0.5, (.5, .5, 0, 0)), (1, (0, 1, 0, 0)), (2, (.1, .2, .3, .4)), (2.9, (0, 0, .1, .9)))
    for mean, weights in patterns if k <= 64 else patterns[2:]:
        L = rng.choice([0, 1, 2, 3], size=int(1.1 * NNZ / mean), p=weights)
        for cols in (900, 40_000 if k <= 64 else 12_000):
            A = wl.csr_from_lengths(L, cols, seed=k)
            assert A.nnz >= 1536 * 256
            Bh = wl.dense_uniform(cols * k, 3, wl.S_B).reshape(cols, k)
            ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
            for pad in (1, 16):
                got = product(A, cols, Bh, k, 256, pad=pad)
                ok, worst = oracle.within_tolerance(got, ref, mag)
                assert ok, "mean %g cols %d pad %d: %.3g of the bar" % (mean, cols, pad, worst)


def test_narrow_rows_take_no_longer_than_wide_ones():
    """Two million rows of one entry: rows of 8 and 12 columns share 64-byte pieces of C and rows of 16 fill them.  Stored past the L2 one
    by one the former took 1.7 to 2.2 times as long as the latter (87 and 114 us against 51)."""
    A = wl.csr_from_lengths(np.ones(2_000_000, dtype=np.int64), 8000, seed=1)
    pos, crd, vals = dev(A.pos), dev(A.crd), dev(A.vals)
    ws = psk.workspace(psk.PSK_OP_SPMM_CSR, A.rows, A.nnz, k=16)
    took = {}
    for k in (8, 12, 16):
        B = dev(wl.dense_uniform(8000 * k, 3, wl.S_B).reshape(8000, k))
        C = torch.empty((A.rows, k), device="cuda")
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                psk.psk_spmm_csr(A.rows, 8000, A.nnz, pos, crd, vals, B, C, ws=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[k] = min(times)
    print(took, flush=True)
    assert max(took[8], took[12]) <= 1.35 * took[16]


@pytest.mark.parametrize("k,per", [(6, 16), (16, 3), (32, 16), (40, 300), (64, 16), (100, 16), (200, 300)])
def test_offsets_beyond_32_bits(k, per):
    """B as rows far apart: from 2^30 floats of cols * ldb on the byte offsets into B don't fit 32 bits, and the end of a row is marked in
    the column instead of in the offset.  One row stride on either side, the last rows of B referred to."""
    cols = 1100
    A = wl.csr_from_lengths(np.full((2000 * 256) // per + 5, per), cols, seed=k)
    assert A.crd.max() == cols - 1 and A.nnz >= 1536 * 256
    Bh = wl.dense_uniform(cols * k, 5, wl.S_B).reshape(cols, k)
    ref, mag = oracle.spmm_csr(A.pos, A.crd, A.vals, Bh)
    most = (2 ** 32 - 1) // 4 // cols
    buf = torch.empty(cols * (most + 1), device="cuda")
    for ld in (most, most + 1):
        B = buf[:cols * ld].view(cols, ld)[:, ld - k:]            # the last columns: offsets up to the end of the buffer
        B.copy_(dev(Bh))
        C = torch.full((A.rows, k), float("nan"), device="cuda")
        print("spmm wave offsets k", k, "ld", ld, flush=True)
        psk.psk_spmm_csr(A.rows, cols, A.nnz, dev(A.pos), dev(A.crd), dev(A.vals), B, C, tile=256)
        torch.cuda.synchronize()
        ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, mag)
        assert ok, "k %d ld %d: %.3g of the bar" % (k, ld, worst)
