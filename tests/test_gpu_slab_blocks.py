"""The analysis step of the column-slab path works in blocks of 2048 positions and decides inside a block where the pairs of
its rows start and end; rows that cross blocks are decided from counts.  The structure is compared bit for bit with the
oracle's where that can go wrong: sizes around a block, rows that cross one or many blocks with and without entries of a
slab in between, the largest number of slabs of this path, long runs of empty rows, operands without 16-byte alignment."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402

BLOCK = 2048


def dev(a, shift):
    """The array on the GPU, `shift` elements behind an aligned address."""
    t = torch.empty(a.size + shift, dtype=torch.from_numpy(a[:0]).dtype, device="cuda")
    t[shift:] = torch.from_numpy(a).cuda()
    return t[shift:]


def check(pos, crd, cols, f64, shift=0):
    pos, crd = np.asarray(pos, dtype=np.int32), np.asarray(crd, dtype=np.int32)
    vals = wl.dense_uniform(crd.size, 5, wl.S_VALS).astype(np.float64 if f64 else np.float32)
    rows = pos.size - 1
    S = (psk.psk_slab_build_csr_f64 if f64 else psk.psk_slab_build_csr)(
        rows, cols, crd.size, dev(pos, 0), dev(crd, shift), dev(vals, shift))
    O = oracle.slab_build(rows, cols, pos, crd, vals, W=16352 if f64 else 32736, f64=f64)
    d = S.desc
    assert (d.nslots, d.npairs, d.nq, d.nslabs) == (O.nslots, O.npairs, O.nq, (cols + O.W - 1) // O.W)
    for arr in ("slab_chunk", "chunk_pair", "qpos", "qidx"):
        assert np.array_equal(S.array(arr).cpu().numpy(), getattr(O, arr)), arr
    assert np.array_equal(S.array("scol").cpu().numpy().view(np.uint16), O.scol)
    assert np.array_equal(S.array("svals").cpu().numpy().view(np.uint8), O.svals.view(np.uint8))
    assert np.array_equal(S.array("qtile_row").cpu().numpy(), oracle.partition(O.qpos, d.tile))


def cut(lengths):
    return np.concatenate([[0], np.cumsum(lengths)])


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n", [BLOCK - 1, BLOCK, BLOCK + 1, 3 * BLOCK - 1, 3 * BLOCK])
def test_row_borders_around_blocks(n, f64):
    rng = np.random.default_rng(n)
    cols = 200_000
    for lengths in ([n], [1] * n, [BLOCK - 1, n - BLOCK + 1], [n - 3, 0, 3], [n // 3, n - n // 3 - 1, 1]):
        check(cut(lengths), rng.integers(0, cols, n), cols, f64)


@pytest.mark.parametrize("f64", [False, True])
def test_rows_over_many_blocks_with_gaps_in_a_slab(f64):
    # one row over five blocks: slab 0 only in its first and last block, slab 1 only in its first, slab 2 only in a middle one
    W, n = (16352 if f64 else 32736), 5 * BLOCK + 100
    crd = np.full(n, 3 * W + 7)
    crd[50:60], crd[n - 150:n - 140] = 3, 5
    crd[60:70] = W + 1
    crd[2 * BLOCK + 9] = 2 * W
    for lengths in ([n], [55, n - 55], [40, n - 180, 140], [n - 145, 145]):
        check(cut(lengths), crd, 4 * W, f64)


@pytest.mark.parametrize("nslabs", [1, 2, 64, 65, 128, 129, 255, 256, 257])
def test_number_of_slabs(nslabs):
    rng = np.random.default_rng(nslabs)
    cols = nslabs * 32736 - 1
    lengths = rng.choice([0, 1, 2, 5, 40, 3000], size=400, p=[.2, .3, .2, .2, .09, .01])
    n = int(lengths.sum())
    check(cut(lengths), rng.integers(0, cols, n), cols, False)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_operands_and_long_runs_of_empty_rows(shift):
    rng = np.random.default_rng(shift)
    lengths = np.zeros(70_000, dtype=np.int64)
    lengths[[0, 3, 20_000, 45_000, 69_999]] = [BLOCK - 5, 9, 30, BLOCK, 1]
    n = int(lengths.sum())
    check(cut(lengths), rng.integers(0, 100_000, n), 100_000, shift == 2, shift)
