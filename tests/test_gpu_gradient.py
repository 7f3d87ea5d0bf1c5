"""The one-launch gradient of dense features at the edges of its layout: columns around every switch of the number of
wavefronts that share a row and of blocks that share a row, rows around what a block holds at a time, ragged shards
and the first length that takes the two-kernel form; the gradients of two points against fp64."""
import numpy as np
import pytest

from test_gpu_parity import _cuda, _eng

pytestmark = pytest.mark.gpu

SHAPES = [(3, 1, 5), (2, 20, 300), (4, 256, 128), (3, 257, 129), (2, 511, 65), (2, 513, 33), (3, 1024, 31), (2, 1025, 17), (5, 2048, 16),
          (3, 2049, 40), (2, 5003, 203), (1, 20000, 9), (40, 4099, 33), (70, 65536, 5), (2, 131072, 3), (2, 131073, 3), (600, 40, 7)]


@pytest.mark.parametrize("n,d,rows", SHAPES)
def test_gradient_at_the_edges_of_its_layout(n, d, rows):
    rng = np.random.default_rng(d * 7 + rows)
    cnt = rows - rng.integers(0, max(1, rows // 2), size=n)
    cnt[0] = rows
    check_gradient(n, d, rows, cnt, rng)


# one shard of `rows` rows among shards of `short`: chunks by a table; chunk counts around what one block adds up; blocks with
# one group of wavefronts
@pytest.mark.parametrize("n,d,rows,short", [(40, 300, 9000, 3), (100, 2049, 3000, 5), (3, 65536, 300, 1), (5, 16384, 700, 40), (300, 17, 5000, 8),
                                            (1, 2048, 4000, 0), (1, 2048, 256, 0), (1, 2048, 257, 0), (1, 2048, 272, 0), (1, 2048, 273, 0),
                                            (2, 3, 40000, 39999), (1500, 30, 8, 8), (1100, 700, 17, 1), (1, 5003, 2000, 0)])
def test_gradient_of_a_long_shard_among_short_ones(n, d, rows, short):
    rng = np.random.default_rng(d * 11 + rows)
    cnt = np.full(n, short)
    cnt[n // 2] = rows
    check_gradient(n, d, rows, cnt, rng)


@pytest.mark.parametrize("n,d,rows,short", [(3, 2049, 40, 40), (5, 5003, 203, 150), (3, 65536, 300, 1), (1, 131072, 20, 0), (90, 4099, 5, 5),
                                            (1, 16384, 900, 0)])
def test_gradient_where_blocks_do_not_wait_for_each_other(n, d, rows, short):
    """A chunk whose blocks were not all running at once is formed by one of them."""
    cnt = np.full(n, short)
    cnt[n // 2] = rows
    check_gradient(n, d, rows, cnt, np.random.default_rng(d * 13 + rows), _eng().FLAG_NO_WAIT)


# chunk counts around those that one group of wavefronts adds, that several share, and that are added at once: 8, 9, 16, 17, 32, 33 chunks
# and more, whose sixteens are eight, nine and seventeen sums, in blocks of eight, four and two groups (128, 64 and 32 rows a chunk)
# and of one
@pytest.mark.parametrize("n,d,rows", [(2, d, held * c + more) for d, held in ((100, 128), (300, 64), (1000, 32), (2048, 16))
                                      for c, more in ((1, 0), (8, 0), (8, 1), (16, 0), (16, 1), (32, 0), (32, 1), (64, 1))]
                         + [(1, 100, 16384), (1, 100, 16385), (1, 300, 4097), (1, 1024, 1024), (1, 1024, 1025), (1, 1024, 17000), (1, 700, 2000)])
def test_gradient_around_the_counts_of_partial_sums(n, d, rows):
    check_gradient(n, d, rows, np.full(n, rows), np.random.default_rng(d * 19 + rows))


# lengths with rows that begin on lines (multiples of 32: blocks take turns of columns) and without, a few columns in the last turn
# or part; the last three, of one length each, have more features than are kept in the cache, as many as are, and rows off the lines
@pytest.mark.parametrize("n,d,rows", [(3, 2080, 40), (3, 2303, 40), (3, 2304, 17), (2, 4064, 33), (2, 4112, 33), (1, 131040, 20), (1, 131056, 20),
                                      (100, 131072, 7), (80, 131072, 7), (100, 130000, 7)])
def test_gradient_of_rows_on_and_off_the_lines(n, d, rows):
    check_gradient(n, d, rows, np.full(n, rows), np.random.default_rng(d * 17 + rows))


def check_gradient(n, d, rows, cnt, rng, flags=0):
    E = _eng()
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    A = rng.standard_normal((int(off[-1]), d), dtype=np.float32)
    y = np.where(rng.random(int(off[-1])) < 0.5, 1.0, -1.0).astype(np.float32)
    x0 = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    eng = E.AdaCGD(n=n, d=d, gamma=0.3, lam=0.1, worker_levels=[(E.TOPK, max(1, d // 10)), (E.TOPK, d)], zeta_worker=0.0,
                   master_levels=[], grad_mode=E.GRAD_LOGISTIC, A=_cuda(A), labels=_cuda(y), shard_offsets=off, x0=_cuda(x0),
                   flags=E.FLAG_ANY_LEVEL_ORDER | flags)
    for step in range(4):        # (both sets of what blocks meet at are used twice)
        if step:
            eng.step()
        x = eng.state(E.F_X).astype(np.float64)
        got = eng.state(E.F_GRAD).reshape(n, d)
        for i in range(n):
            a = A[off[i]:off[i + 1]].astype(np.float64)
            yi = y[off[i]:off[i + 1]].astype(np.float64)
            s = -yi / (1.0 + np.exp(yi * (a @ x))) / len(yi)
            want = s @ a + 2 * np.float64(np.float32(0.1)) * x / (1 + x * x) ** 2
            # fp64 sums rounded once: half a unit of the result, and what the sums themselves may lose (2^-52 a term)
            bound = np.abs(want) * 2.0 ** -23 + (np.abs(s) @ np.abs(a)) * (d + len(yi)) * 2.0 ** -52
            assert (np.abs(got[i] - want) <= bound).all(), (n, d, rows, step, i)
    eng.close()
