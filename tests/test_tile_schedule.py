"""Host-side check of the tiled GEMM kernels' work split (no GPU): the library replays the schedule its
persistent workgroups walk, and every (row panel, 64-column strip, K group) must be covered exactly once."""
import ctypes as C

import numpy as np
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2603_16590_amd import binding
    return binding.lib


def _schedule(lib, M, N, K, cus, glu, ksplit, a8=False):
    mode = int(glu) + 2 * int(a8)
    n = lib.batq_debug_tile_schedule(M, N, K, cus, mode, int(ksplit), None, 0)
    assert n > 0
    buf = (C.c_int * (7 * n))()
    assert lib.batq_debug_tile_schedule(M, N, K, cus, mode, int(ksplit), buf, n) == n
    return np.frombuffer(buf, dtype=np.int32).reshape(n, 7).copy()


def _check(lib, M, N, K, cus, glu, ksplit):
    t = _schedule(lib, M, N, K, cus, glu, ksplit)
    wg, m0, n0, nj, part, g0, ng = t.T
    panels, groups = -(-M // 256), -(-K // 256)
    unit = 128 if glu else 64
    strips = -(-N // unit) * (unit // 64)
    workers = 8 * max(1, cus // 8)
    assert wg.min() >= 0 and wg.max() < workers
    assert np.all(m0 % 256 == 0) and np.all(m0 < panels * 256)
    assert np.all(n0 % unit == 0) and np.all((nj >= 1) & (nj <= 4)) and np.all(n0 // 64 + nj <= strips)
    if glu:
        assert np.all(nj % 2 == 0)
    assert np.all(ng >= 1) and np.all(g0 >= 0) and np.all(g0 + ng <= groups)
    cover = np.zeros((panels, strips, groups), dtype=np.int32)
    for i in range(len(t)):
        cover[m0[i] // 256, n0[i] // 64:n0[i] // 64 + nj[i], g0[i]:g0[i] + ng[i]] += 1
    assert np.all(cover == 1), (M, N, K, cus, glu, ksplit, int(cover.min()), int(cover.max()))
    nparts = part.max() + 1
    if nparts > 1:
        assert ksplit and not glu and nparts <= 8
        assert np.all(ng >= 12)                                   # a part keeps at least 12 K groups
        assert panels * (strips // (unit // 64)) * 2 <= workers   # only when at most half the workgroups had a strip
        for p in range(nparts):                                   # same K range for every tile of a part
            assert len(set(zip(g0[part == p], ng[part == p]))) == 1
    # equal shares: strips x K groups per workgroup differ by at most one unit's worth
    load = np.zeros(workers, dtype=np.int64)
    np.add.at(load, wg, (nj // (unit // 64)).astype(np.int64))
    assert load.max() - load.min() <= 1
    return t


def test_headline_shapes(lib):
    # cfg2: 1792 strips over 256 workgroups = 7 each, as a 4-strip and a 3-strip tile
    t = _check(lib, 2048, 14336, 4096, 256, False, True)
    assert len(t) == 512 and sorted(set(t[:, 3])) == [3, 4] and t[:, 4].max() == 0
    # cfg3: one 256 x 256 tile per workgroup
    t = _check(lib, 4096, 4096, 14336, 256, False, True)
    assert len(t) == 256 and np.all(t[:, 3] == 4) and np.all(t[:, 6] == 56)
    # down projection at 256 rows: 64 strips, K cut into 4 parts of 14 groups
    t = _check(lib, 256, 4096, 14336, 256, False, True)
    assert t[:, 4].max() == 3 and np.all(t[:, 6] == 14) and len(t) == 256
    t = _check(lib, 256, 4096, 14336, 256, False, False)
    assert t[:, 4].max() == 0 and len(t) == 64
    # gated gate/up GEMM of cfg2's block: tiles 2 or 4 strips wide
    t = _check(lib, 2048, 28672, 4096, 256, True, True)
    assert sorted(set(t[:, 3])) == [2, 4]


def test_column_bands_follow_the_tile_rounds(lib):
    """The workgroups of one XCD (workgroup index mod 8) own a compact block of the output.  Its A rows are streamed
    once per tile round, so many rounds call for few bands (a tall-narrow block would re-read much of A every round):
    cfg4's ten rounds give every XCD 1024 rows and all columns; cfg3's single round the 1024 x 2048 blocks that
    minimise rows + columns; cfg2's two rounds 1024 x 3584."""
    for (M, K, N), rows, cols in (((8192, 3584, 18944), 1024, 18944), ((4096, 14336, 4096), 1024, 2048),
                                  ((2048, 4096, 14336), 1024, 3584)):
        t = _check(lib, M, N, K, 256, False, False)
        for x in range(8):
            mine = t[t[:, 0] % 8 == x]
            r = mine[:, 1].max() + 256 - mine[:, 1].min()
            c = (mine[:, 2] + 64 * mine[:, 3]).max() - mine[:, 2].min()
            assert (r, c) == (rows, cols), ((M, K, N), x, r, c)


def test_workgroups_of_an_xcd_take_turns_with_the_narrow_tiles(lib):
    """A run of strips is cut into tiles of two widths one strip apart.  If every workgroup put the wide ones first,
    all would reach their epilogues together and the chip would write its output in bursts; so workgroup i of an XCD
    puts i % (number of narrow tiles + 1), at most 3, narrow tiles in front.  Workgroups 8 apart inside an XCD stream
    the same weight columns and must stay in step."""
    def widths(t, b):
        return [int(x[3]) for x in t if x[0] == b]
    t = _check(lib, 8192, 18944, 3584, 256, False, False)       # cfg4: 37 strips per workgroup = 7 x 4 + 3 x 3
    for x in (0, 5):
        assert widths(t, x) == [4] * 7 + [3] * 3
        assert widths(t, x + 8) == [3] + [4] * 7 + [3] * 2
        assert widths(t, x + 16) == [3] * 2 + [4] * 7 + [3]
        assert widths(t, x + 24) == [3] * 3 + [4] * 7
        assert widths(t, x + 32) == widths(t, x)
    for b in range(256):                                       # same columns (8 workgroups apart in the XCD): same order
        i = b >> 3
        if i + 8 < 32:
            assert widths(t, b) == widths(t, b + 64)
    t = _check(lib, 2048, 14336, 4096, 256, False, False)       # cfg2: 7 strips = 4 + 3
    assert widths(t, 0) == [4, 3] and widths(t, 8) == [3, 4] and widths(t, 16) == [4, 3] and widths(t, 24) == [3, 4]
    t = _check(lib, 4096, 4096, 14336, 256, False, False)       # cfg3: one tile each, nothing to reorder
    assert all(widths(t, b) == [4] for b in range(256))


def test_random_shapes(lib):
    rng = np.random.default_rng(0)
    for _ in range(300):
        M = int(rng.integers(65, 5000))
        N = int(rng.integers(1, 20000))
        K = 32 * int(rng.integers(1, 700))
        cus = int(rng.choice([8, 40, 64, 256, 304]))
        glu = bool(rng.integers(0, 2))
        if glu:
            N = 64 * max(1, N // 64)
        _check(lib, M, N, K, cus, glu, bool(rng.integers(0, 2)))
    # few-strip, long-K corner: every split factor from 2 to 8
    seen = set()
    for N in (64, 128, 192, 640, 1024, 2048, 4096):
        for K in (6144, 8192, 14336, 32768):
            for M in (65, 256, 257, 700):
                t = _check(lib, M, N, K, 256, False, True)
                seen.add(int(t[:, 4].max()) + 1)
    assert seen >= {1, 2, 4, 8}, seen


def test_invalid_arguments(lib):
    assert lib.batq_debug_tile_schedule(64, 128, 256, 256, 0, 0, None, 0) == -1     # M <= 64 takes the small-M kernel
    assert lib.batq_debug_tile_schedule(100, 128, 100, 256, 0, 0, None, 0) == -1
    assert lib.batq_debug_tile_schedule(100, 96, 256, 256, 1, 0, None, 0) == -1     # gated output needs N % 64 == 0
    assert lib.batq_debug_tile_schedule(100, 128, 256, 256, 0, 0, None, 5) == -1


@pytest.mark.parametrize("M,N,glu", [(700, 8192, False), (3449, 2963, False), (5327, 1786, False), (2300, 14336, False),
                                     (2720, 5802, False), (1290, 17749, False), (5293, 6075, False), (2500, 4096, False),
                                     (700, 16384, True), (2500, 8192, True)])
def test_no_share_reaches_into_the_next_run(lib, M, N, glu):
    """A share that crosses from one row panel of a band into the next takes an extra tile, and the launch waits for it:
    where the shares come in two sizes every workgroup gets as few tiles as the larger size needs."""
    t = _check(lib, M, N, 4096, 256, glu, False)
    units = (-(-M // 256)) * (-(-N // (128 if glu else 64)))
    assert units % 256 and units > 256
    most = -(-(units // 256 + 1) // (2 if glu else 4))
    assert np.bincount(t[:, 0]).max() == most


def _bands(t):
    """Column bands of a schedule: in share order the row panels of one band follow those of the one before."""
    share = (t[:, 0] % 8) * (256 // 8) + t[:, 0] // 8
    m0 = t[np.argsort(share, kind="stable"), 1]
    return 1 + int(np.sum(np.diff(m0) < 0))


def _band_bytes(M, N, glu):
    """Bytes the L2s pull with 1, 2, 4 and 8 bands, in the model of the work split: rounds x bands x M + 8 / bands x N."""
    units = -(-M // 256) * -(-N // (128 if glu else 64))
    per = -(-units // 256)
    rounds = -(-per // 4) if per > 4 else 1
    return {b: rounds * b * M + 8 / b * N for b in (1, 2, 4, 8) if b <= -(-N // (128 if glu else 64))}, per


@pytest.mark.parametrize("M,K,N,a8,most", [
    (1664, 4096, 7120, False, 2.6), (656, 1024, 16668, False, 2.6), (1529, 1024, 8237, False, 2.6),
    (1520, 1024, 8202, True, 1.4), (2121, 1024, 5648, True, 1.4), (1400, 1024, 10448, True, 1.4)])
def test_bytes_given_for_whole_shares_are_bounded_on_ragged_rows(lib, M, K, N, a8, most):
    """Output rows that do not start on whole lines, shares of three and four strips, short K: the second tile of a share costs
    less than the bytes of a band count that avoids it."""
    cost, _ = _band_bytes(M, N, False)
    assert cost[_bands(_schedule(lib, M, N, K, 256, False, False, a8))] < most * min(cost.values())


def test_fewest_bytes_where_every_band_count_leaves_costly_shares(lib):
    """Where no band count keeps the shares inside their runs, more (or wider) bands only move more bytes: the cheapest count
    serves; with 8-bit codes and shares of up to three strips a single band, which has the fewest runs."""
    rng = np.random.default_rng(11)
    shapes = [(765, 16344, False), (768, 16384, False), (1536, 8192, False), (3072, 4096, False), (6144, 2048, False),
              (2393, 6458, False), (7363, 1607, False), (2446, 12928, True), (16500, 896, False), (20000, 512, False),
              (20000, 768, False), (32768, 512, False)]
    for _ in range(600):
        glu = bool(rng.integers(0, 4) == 0)
        shapes.append((int(np.exp(rng.uniform(np.log(300), np.log(20000)))),
                       64 * int(np.exp(rng.uniform(np.log(8), np.log(300)))) - (0 if glu else int(rng.integers(0, 64))), glu))
    hit = {False: 0, True: 0}
    for M, N, glu in shapes:
        cost, per = _band_bytes(M, N, glu)
        if -(-M // 256) * -(-N // (128 if glu else 64)) <= 256:
            continue                                        # a strip or less per workgroup: no share has two
        for a8 in (False, True):
            t = _schedule(lib, M, N, 4096, 256, glu, False, a8)
            if np.bincount(t[:, 0]).max() <= -(-per // (2 if glu else 4)):
                continue                                    # no share takes more tiles than the largest alone needs
            bands, least = _bands(t), min(cost.values())
            hit[a8] += 1
            assert cost[bands] == least or (a8 and per <= 3 and bands == 1), (M, N, glu, a8, bands, cost)
    assert hit[False] >= 50 and hit[True] >= 50, hit
