"""Rows of any width through query, insert and update: row lists whose chunks fill a wave load, miss it
by one, or split a row over two of them; batches below, at and above the query's launch shapes.

Three modes of the query: "plain"; "quiet", the default mode with no writer at work (rows validated by the writers'
counts); "held", the default mode while a writer holds a set (here one that no key of the batch falls into), so that
every row goes by its set's sequence word."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from harness import SENTINEL, DeviceCache  # noqa: E402
from oracle import OracleCache  # noqa: E402
from paper_2210_08804_amd import binding as B  # noqa: E402
from paper_2210_08804_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def _hold_a_set(gc, oc, space):
    """Holds a set as a writer would; returns the keys below `space` that fall into the others."""
    sets = np.array([oc.set_of(k) for k in range(space)])
    spare = int(sets[0])
    B.hps_cache_debug_set_seq(gc.h, spare, 1)
    started, finished = B.hps_cache_debug_writers(gc.h)
    assert started == finished + 1
    return np.nonzero(sets != spare)[0].astype(np.int64)


def _compare(gc, oc, keys, d):
    exp = np.full((len(keys), d), SENTINEL, dtype=np.uint32)
    _, omi, _ = oc.query(keys, exp)
    out, mi, mk = gc.query(keys)
    assert (mi == omi).all() and (mk == keys[omi]).all()
    assert (out == exp).all()


@pytest.mark.parametrize("mode", ["plain", "quiet", "held"])
@pytest.mark.parametrize("d", [4, 8, 12, 28, 32, 36, 64, 68, 96, 124, 132, 192, 252, 260, 320, 512, 516, 1020, 1024])
def test_row_widths(d, mode):
    S, W, n_keys = 2039, 8, 1200            # no set gets more than W keys
    keys = np.arange(n_keys, dtype=np.int64) * 7 + 1
    rows = inputs.backing_rows(keys, d)
    with DeviceCache(S * W, W, d, concurrent_writers=mode != "plain") as gc:
        oc = OracleCache(S * W, W, d)
        for lo in range(0, n_keys, 401):
            gc.insert(keys[lo:lo + 401], rows[lo:lo + 401])
            oc.insert(keys[lo:lo + 401], rows[lo:lo + 401])
        upd = keys[::3].copy()
        gc.update(upd, inputs.backing_rows(upd, d, version=1))
        oc.update(upd, inputs.backing_rows(upd, d, version=1))
        rng = np.random.Generator(np.random.PCG64(d))
        others = _hold_a_set(gc, oc, 9 * n_keys) if mode == "held" else None
        for n in (1, 7, 63, 65, 1000):
            _compare(gc, oc, rng.integers(0, 9 * n_keys, size=n, dtype=np.int64) if others is None else rng.choice(others, n), d)
        oc.close()


@pytest.mark.parametrize("mode", ["plain", "quiet", "held"])
@pytest.mark.parametrize("d,n", [(16, (1 << 14) - 1), (16, 1 << 14), (16, (1 << 18) + 3), (32, (1 << 17) + 1), (32, 270001), (64, (1 << 16) + 7),
                                 (64, 270001), (96, 43691), (160, 20001), (128, 4095), (128, 4097), (128, 10239), (128, 10240), (128, 28673),
                                 (128, 57345), (128, 16385), (256, 16384), (320, 13107), (320, 60001)])
def test_shapes_by_batch_and_width(d, n, mode):
    """Both sides of every line between two launch shapes."""
    S, W, n_keys = 8191, 8, 4000
    keys = np.arange(n_keys, dtype=np.int64) * 5
    rows = inputs.backing_rows(keys, d)
    with DeviceCache(S * W, W, d, concurrent_writers=mode != "plain") as gc:
        oc = OracleCache(S * W, W, d)
        gc.insert(keys, rows)
        oc.insert(keys, rows)
        rng = np.random.Generator(np.random.PCG64(n))
        others = _hold_a_set(gc, oc, 6 * n_keys) if mode == "held" else None
        _compare(gc, oc, rng.integers(0, 6 * n_keys, size=n, dtype=np.int64) if others is None else rng.choice(others, n), d)
        oc.close()


@pytest.mark.parametrize("W,d", [(1, 12), (1, 16), (4, 60), (4, 64), (8, 60), (8, 64), (8, 124), (8, 192), (8, 256), (8, 260), (8, 320), (8, 516), (16, 60),
                                 (16, 64), (16, 260), (32, 124), (32, 128), (32, 260), (64, 128), (64, 260)])
def test_updates_on_both_sides_of_their_switches(W, d):
    """16 keys to a wave below 32,768 of them and, for rows long enough, up to 49,152, else 64; there each lane searches its own set in a
    dump's order and where few lanes search, W lanes search it otherwise.  Cached keys, absent ones and keys given twice (with the same
    row); rows of less than a wave load, of one and of several."""
    S = (1 << 16) // W
    rng = np.random.Generator(np.random.PCG64(1000 * W + d))
    with DeviceCache(S * W, W, d) as gc:
        oc = OracleCache(S * W, W, d)
        pool = np.arange(1, S * W, dtype=np.int64)
        gc.insert(pool, inputs.backing_rows(pool, d))
        gk, gctr, gv = gc.export()
        oc.load_state(gk, gctr, gv)
        cached = gk[gk != -(1 << 63)]
        slots = np.resize(cached, 70001)
        mixed = rng.permutation(np.concatenate([cached, cached[:3000], pool[:20000] + 10 ** 7]))
        for version, keys in enumerate([slots[:32767], slots[:32768], slots[:49152], slots[:49153], slots,
                                        mixed[:32768], np.resize(mixed, 49152), np.resize(mixed, 49153)], 1):
            rows = inputs.backing_rows(keys, d, version=version)
            gc.update(keys, rows)
            oc.update(keys, rows)
            gk2, gctr2, gv2 = gc.export()
            assert (gk2 == gk).all() and (gctr2 == gctr).all() and (gv2 == np.array(oc.vals)).all()
        oc.close()


@pytest.mark.parametrize("n", [5000, 33000])
@pytest.mark.parametrize("d", [4, 60, 64, 124, 192, 256, 260])
def test_writers_by_width(d, n):
    """Rows that divide a wave's lanes and rows that do not, up to and above one wave load, in inserts on both sides of their
    switch and updates of half as many rows, 16 keys to a wave."""
    S, W = 131071, 8                         # no set gets more than W keys
    keys = np.arange(n, dtype=np.int64) * 3 + 1
    with DeviceCache(S * W, W, d) as gc:
        oc = OracleCache(S * W, W, d)
        for version, write in ((0, "insert"), (1, "update")):
            batch = keys[version::2].copy() if version else keys
            rows = inputs.backing_rows(batch, d, version=version)
            getattr(gc, write)(batch, rows)
            getattr(oc, write)(batch, rows)
        _compare(gc, oc, keys, d)
        oc.close()


@pytest.mark.parametrize("n", [1, 63, 65, 49152, 49153])
@pytest.mark.parametrize("W", [1, 2, 8, 32, 64])
def test_update_finds_its_keys_in_any_set(W, n):
    """16 and 64 keys to a wave on both sides of the switch between them: cached keys in random order, next to each other in slot
    order, given twice (with the same row), absent ones and the reserved values."""
    S, d = 1021, 8
    rng = np.random.Generator(np.random.PCG64(n + W))
    pool = np.arange(1, S * W, dtype=np.int64)
    rows = inputs.backing_rows(pool, d)
    with DeviceCache(S * W, W, d) as gc:
        oc = OracleCache(S * W, W, d)
        gc.insert(pool, rows)
        gk, gctr, gv = gc.export()
        oc.load_state(gk, gctr, gv)
        cached = gk[gk != -(1 << 63)]
        keys = np.concatenate([cached, rng.choice(cached, 30000), pool + 10 ** 7, np.array([-(1 << 63), -(1 << 63) + 1] * 20, dtype=np.int64)])
        for order in ("slots", "random"):
            k = np.resize(keys, n) if order == "slots" else rng.choice(keys, n)
            r = inputs.backing_rows(k, d, version=1 + (order == "random"))
            gc.update(k, r)
            oc.update(k, r)
            gk2, gctr2, gv2 = gc.export()
            assert (gk2 == gk).all() and (gctr2 == gctr).all() and (gv2 == np.array(oc.vals)).all()
        oc.close()
