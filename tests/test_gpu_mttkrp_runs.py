"""MTTKRP in runs of leaves per group of lanes: the narrow widths, the chunks of 32 columns of a large D, fibers that cover many
runs, slices that end at the border of a run, a wave's share and a tile, more empty slices than 16 bits number, and the table
of the cut for few, many and very many tiles.  Bar: |got - ref| <= 1e-5 * sum |b c d| + 1e-30; tables bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_mttkrp_groups import check, dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


@pytest.mark.parametrize("j", [4, 5, 7, 8, 9, 12, 16, 24, 48, 64, 66, 96, 97, 128, 129, 160, 261])
def test_widths(j):
    rng = np.random.default_rng(j)
    fps = rng.integers(0, 5, size=300)
    leaves = rng.choice([0, 1, 2, 15, 16, 17, 33, 400], size=int(fps.sum()))
    check(fps, leaves, (300, 250, 700), j, 256)
    check([1, 1, 2, 1], [2048, 8, 600, 2040, 3], (4, 30, 3000), j, 2048, pad=0)


@pytest.mark.parametrize("j", [32, 64, 96])
def test_chunks_of_a_large_factor_matrix(j):
    """Rows of D that begin 128-byte lines and D above 6 MiB; a few hundred tiles, so not the chunks of few tiles."""
    rng = np.random.default_rng(j)
    fps = rng.integers(1, 6, size=3000)
    check(fps, rng.choice([1, 3, 40], size=int(fps.sum())), (3000, 900, (6 << 18) // j + 100), j, 256, pad=0)


def test_runs_of_empty_slices():
    fps = np.concatenate([[2, 3, 1], np.zeros(70_000, dtype=int), [1, 2], np.zeros(300, dtype=int), [4] * 40])
    check(fps, np.full(int(fps.sum()), 9), (fps.size, 250, 700), 8, 2048)


@pytest.mark.parametrize("tile", [1, 7, 2048])
def test_table(tile):
    """One, four and 64 lanes per entry (up to 12 000 and up to 100 000 tiles)."""
    rng = np.random.default_rng(3)
    fps = rng.integers(0, 6, size=16_000)
    T = wl.csf3_from_lengths(fps, rng.choice([0, 1, 2, 9], size=int(fps.sum())), (16_000, 500, 700), seed=1)
    n = psk.psk_num_tiles(T.nnz, tile)
    assert (n > 100_000) if tile == 1 else (12_000 < n < 100_000 if tile == 7 else n < 12_000)
    s, f = psk.psk_partition_csf3(dev(T.pos_k), dev(T.pos_l), T.nnz, tile)
    ref_s, ref_f = oracle.partition_csf3(T.pos_k, T.pos_l, tile)
    assert (s.cpu().numpy() == ref_s).all() and (f.cpu().numpy() == ref_f).all()
