"""MTTKRP where its kernels change over: numbers of columns around the group widths and chunks, tiles whose leaves divide evenly
among the groups and tiles that do not (the last one), fibers and slices that end at a group's, a wave's or a tile's border,
operands whose rows are not aligned, and the sizes from which a product goes to the kernel of one to four columns per lane.
Bar: |got - ref| <= 1e-5 * sum |b c d| + 1e-30 per element."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2001_00532_amd as psk  # noqa: E402


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(fibers, leaves, dims, j, tile, pad=1, compressed=False):
    T = wl.csf3_from_lengths(np.asarray(fibers), np.asarray(leaves), dims, seed=j + 3, compressed_i=compressed)
    I, K, L = dims
    C = wl.dense_uniform(K * (j + pad), 7, wl.S_B).reshape(K, j + pad)
    D = wl.dense_uniform(L * (j + pad), 8, wl.S_B).reshape(L, j + pad)
    ref, mag = oracle.mttkrp_csf3(T.pos_k, T.crd_k, T.pos_l, T.crd_l, T.vals, C[:, :j], D[:, :j], threads=8)
    rows = T.crd_i if compressed else np.arange(T.nslices)
    want, bar = np.zeros((I, j)), np.zeros((I, j))
    want[rows], bar[rows] = ref, mag
    A = torch.full((I, j + pad), float("nan"), device="cuda")
    psk.psk_mttkrp_csf3(dims, dev(T.crd_i), dev(T.pos_k), dev(T.crd_k), dev(T.pos_l), dev(T.crd_l), dev(T.vals),
                        dev(C)[:, :j], dev(D)[:, :j], A[:, :j], tile=tile)
    torch.cuda.synchronize()
    got = A.cpu().numpy()
    assert np.isnan(got[:, j:]).all(), "columns past j were written"
    ok, worst = oracle.within_tolerance(got[:, :j], want, bar)
    assert ok, "j %d tile %d: %.3g of the bar" % (j, tile, worst)


@pytest.mark.parametrize("j", [16, 17, 20, 31, 32, 33, 36, 47, 48, 49, 63, 64, 65, 100, 128, 130])
def test_columns_and_borders(j):
    rng = np.random.default_rng(j)
    fps = rng.integers(0, 6, size=400)
    check(fps, rng.choice([0, 1, 2, 7, 8, 9, 60], size=int(fps.sum())), (400, 300, 500), j, 256)
    check(fps, rng.choice([1, 8, 16, 64], size=int(fps.sum())), (900, 300, 500), j, 1024, pad=0, compressed=True)
    check([1, 1, 2, 1], [256, 8, 248, 2048, 5], (4, 30, 3000), j, 256, pad=3)


@pytest.mark.parametrize("tile", [0, 256, 512, 1024, 2048])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 4096 + 31])
def test_uneven_last_tiles(n, tile):
    check([1], [n], (1, 5, 5000), 24, tile)
    check([n // 3, n - 2 * (n // 3)], [1] * (n // 3) + [2] * (n // 3) + [1] * (n - 3 * (n // 3)), (2, 5000, 70), 40, tile)


def test_large_factor_matrix():
    rng = np.random.default_rng(5)
    for L in (30_000, 40_000):                 # 64 columns: 7.7 MB and 10.2 MB (few leaves: groups on either side)
        check(np.full(50, 3), rng.integers(1, 40, size=150), (50, 60, L), 64, 0)
        check(np.full(50, 3), rng.integers(1, 40, size=150), (50, 60, L), 52, 256)


@pytest.mark.parametrize("j,pad", [(66, 2), (72, 0), (96, 0), (96, 4), (100, 0), (101, 0), (130, 2), (192, 0), (200, 0), (200, 2), (258, 2)])
def test_many_tiles_above_64_columns(j, pad):
    """1600 tiles: above 64 columns rows of D that begin 128-byte lines (96 and 192 columns without padding) and odd widths
    stay with the groups, the others go to two or four columns per lane."""
    rng = np.random.default_rng(j + pad)
    fps = rng.integers(0, 9, size=6000)
    leaves = rng.choice([0, 1, 2, 15, 60], size=int(fps.sum()))
    leaves[::1000] = 700
    leaves[-1] += max(0, 1600 * 256 - int(leaves.sum()))
    check(fps, np.minimum(leaves, 9000), (6000, 300, 9000), j, 256, pad=pad)
    check(fps, np.minimum(leaves, 9000), (6500, 300, 9000), j, 256, pad=pad, compressed=True)


@pytest.mark.parametrize("j,pad", [(24, 0), (32, 0), (44, 1), (64, 0)])
@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24])
def test_many_leaves_and_a_large_factor(j, pad, n):
    """From 2^24 leaves on, with a D of more than 9 MiB, the wide kernel takes 17 to 64 columns (not 32 that fill a line)."""
    rng = np.random.default_rng(n & 1)
    leaves = rng.integers(0, 110, size=310_000)
    leaves[:200] += 5000
    leaves = np.minimum(leaves, np.maximum(0, n - np.cumsum(leaves) + leaves))
    leaves[7] += n - int(leaves.sum())
    assert int(leaves.sum()) == n and leaves.max() <= 100_000
    check(np.full(31_000, 10), leaves, (31_000, 400, 100_000), j, 0, pad=pad)


@pytest.mark.parametrize("j", [24, 32, 40, 63])
def test_offsets_beyond_32_bits(j):
    """C or D as rows far apart: from 2^30 floats of rows * stride on the byte offsets don't fit 32 bits (another instance of the
    group kernels, whose offsets are handed on as two words).  One row stride on either side for each of the two."""
    n = 1100
    rng = np.random.default_rng(j)
    fps = np.full(200, 3)
    T = wl.csf3_from_lengths(fps, rng.integers(1, 60, size=600), (200, n, n), seed=j)
    assert T.crd_l.max() == n - 1 and T.crd_k.max() >= n - 5
    Ch, Dh = (wl.dense_uniform(n * j, s, wl.S_B).reshape(n, j) for s in (7, 8))
    ref, mag = oracle.mttkrp_csf3(T.pos_k, T.crd_k, T.pos_l, T.crd_l, T.vals, Ch, Dh)
    most = (2 ** 32 - 1) // 4 // n
    buf = torch.empty(n * (most + 1), device="cuda")
    for ld in (most, most + 1):
        far = buf[:n * ld].view(n, ld)[:, ld - j:]
        for which in ("C", "D"):
            far.copy_(dev(Ch if which == "C" else Dh))
            C, D = (far, dev(Dh)) if which == "C" else (dev(Ch), far)
            A = torch.full((200, j), float("nan"), device="cuda")
            print("mttkrp offsets j", j, "ld", ld, which, flush=True)
            psk.psk_mttkrp_csf3((200, n, n), None, dev(T.pos_k), dev(T.crd_k), dev(T.pos_l), dev(T.crd_l), dev(T.vals), C, D, A)
            torch.cuda.synchronize()
            ok, worst = oracle.within_tolerance(A.cpu().numpy(), ref, mag)
            assert ok, "j %d ld %d %s: %.3g of the bar" % (j, ld, which, worst)
