"""Edges of a query's tiles: lengths that are read on the device, whose keys are dealt to the waves sixteen at a time, and
launch shapes at the batch sizes where the rule changes them.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import OracleCache
from paper_2210_08804_amd import binding as B
from paper_2210_08804_amd import inputs
from harness import DeviceCache, SENTINEL

pytestmark = pytest.mark.gpu


def filled(d, policy=0, ways=8, sets=8192):
    """A cache and its oracle with 6,000 keys, which overflow no set; a batch over twice as many."""
    keys = np.arange(6000, dtype=np.int64)
    rows = inputs.backing_rows(keys, d)
    gc, oc = DeviceCache(sets * ways, ways, d, policy=policy), OracleCache(sets * ways, ways, d)
    for k, r in zip(np.array_split(keys, 12), np.array_split(rows, 12)):
        B.hps_cache_insert(gc.h, torch.from_numpy(k).cuda(), torch.from_numpy(r).cuda(), len(k))
        torch.cuda.synchronize()
        oc.insert(k, r)
    return gc, oc


def expected(oc, keys, d):
    out = np.full((len(keys), d), SENTINEL, dtype=np.uint32)
    _, mi, mk = oc.query(keys, out)
    return out, mi, mk


@pytest.mark.parametrize("checked", [True, False])
@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("d,n_max", [(128, 26624), (32, 7000),      # dealt in sixteens, 32 and 18 keys to a wave
                                     (192, 9000), (320, 30000), (1024, 3000), (512, 20000),   # in 16s, 8s, 2s and 4s, whole ones
                                     (128, 5000), (320, 9000)])      # not dealt: 13 and 12 neighbouring keys to a wave
def test_length_on_the_device_at_the_edges_of_the_deal(d, n_max, policy, checked):
    gc, oc = filled(d, policy)
    with gc:
        B.hps_cache_set_concurrent_writers(gc.h, checked)
        keys = np.random.default_rng(5).integers(0, 12000, n_max)
        dk = torch.from_numpy(keys).cuda()
        # one deal, one wave's and one tile's worth of keys with 4, 5 and 7 workers, and the whole batch; each with its neighbours
        for m in sorted({max(0, min(n_max, e + o)) for e in (0, 4, 16, 28, 32, 56, 64, 80, 112, 128, 1024, n_max) for o in (-1, 0, 1)}):
            out = torch.full((n_max, d), 0, dtype=torch.int32, device="cuda")
            out.fill_(SENTINEL)
            mi = torch.full((n_max,), -1, dtype=torch.int32, device="cuda")
            mk = torch.full((n_max,), -1, dtype=torch.int64, device="cuda")
            nm = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            nd = torch.tensor([m], dtype=torch.int32, device="cuda")
            B.hps_cache_query_dn(gc.h, dk, n_max, nd, out.view(torch.float32), mi, mk, nm)
            torch.cuda.synchronize()
            want, wi, wk = expected(oc, keys[:m], d)
            got = out.cpu().numpy().view(np.uint32)
            assert int(nm.item()) == len(wi), m
            assert (got[:m] == want).all() and (got[m:] == np.uint32(SENTINEL)).all(), m
            order = np.argsort(mi.cpu().numpy()[:len(wi)])
            assert (mi.cpu().numpy()[:len(wi)][order] == wi).all() and (mk.cpu().numpy()[:len(wi)][order] == wk).all(), m
            assert (mi.cpu().numpy()[len(wi):] == -1).all(), m


@pytest.mark.parametrize("checked", [True, False])
@pytest.mark.parametrize("d,n", [
    (128, 1), (128, 3264), (128, 3265), (128, 16384), (128, 16385), (128, 30720), (128, 30721), (128, 57344), (128, 57345),
    (512, 4096), (512, 4097), (512, 7681), (512, 28673), (4, 1 << 19), (16, (1 << 19) - 1), (16, (1 << 19) + 705), (32, (1 << 19) + 1), (64, 1 << 19),
    (68, 1 << 19), (1024, 2049),
    (32, 114689), (32, 180225), (16, 245761), (32, 360449), (32, 491521), (64, 114689), (64, 180225)])
def test_batches_where_the_launch_shape_changes(d, n, checked):
    gc, oc = filled(d)
    with gc:
        B.hps_cache_set_concurrent_writers(gc.h, checked)
        keys = np.random.default_rng(n).integers(0, 12000, n)
        out, mi, mk = gc.query(keys)
        # the oracle looks at every key once
        uniq, inv = np.unique(keys, return_inverse=True)
        want, wi, _ = expected(oc, uniq, d)
        missed = np.zeros(len(uniq), dtype=bool)
        missed[wi] = True
        assert (out == want[inv]).all()
        assert (mi == np.flatnonzero(missed[inv])).all() and (mk == keys[missed[inv]]).all()


@pytest.mark.parametrize("checked", [True, False])
@pytest.mark.parametrize("n_max", [8000, 9000, 40000, 90000, 120000, 130000, 200000])
@pytest.mark.parametrize("ways", [4, 32, 64])
def test_dealt_keys_are_searched_in_sets_of_every_width(ways, n_max, checked):
    """Keys per wave that are no multiple of sixteen: its last lanes get theirs by the deal alone.  (512-byte rows, 256 CUs, plain / default
    mode: 20, 22, 32, 51 / 54, 59 (8 workers) / 36, 37 / 39 and 56 / 59 keys per wave;
    of 64 ways 16, 16, 24, 56, 59 / 36, 37 / 39 and 56 / 59.)"""
    d = 128
    # No set gets more of the keys than it has ways, so which of them are cached does not hang on the order within an insert
    # (4 ways over 8,192 sets: some do; over 2^17 sets, which would have 0.05 keys each, five in one are 2e-9 x 2^17 sets).
    gc, oc = filled(d, ways=ways, sets=1 << 17 if ways < 32 else 1024)
    assert np.bincount([oc.set_of(k) for k in range(6000)]).max() <= ways
    with gc:
        B.hps_cache_set_concurrent_writers(gc.h, checked)
        keys = np.random.default_rng(n_max).integers(0, 12000, n_max)
        dk = torch.from_numpy(keys).cuda()
        uniq, inv = np.unique(keys, return_inverse=True)
        rows, wi, _ = expected(oc, uniq, d)
        missed = np.zeros(len(uniq), dtype=bool)
        missed[wi] = True
        rows, missed = torch.from_numpy(rows.view(np.int32))[torch.from_numpy(inv)].cuda(), missed[inv]
        for m in (n_max, n_max - 1, n_max * 3 // 4, n_max // 3):
            out = torch.full((n_max, d), 0, dtype=torch.int32, device="cuda")
            out.fill_(SENTINEL)
            mi = torch.full((n_max,), -1, dtype=torch.int32, device="cuda")
            mk = torch.full((n_max,), -1, dtype=torch.int64, device="cuda")
            nm = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            nd = torch.tensor([m], dtype=torch.int32, device="cuda")
            B.hps_cache_query_dn(gc.h, dk, n_max, nd, out.view(torch.float32), mi, mk, nm)
            torch.cuda.synchronize()
            want = np.flatnonzero(missed[:m])
            assert int(nm.item()) == len(want), m
            assert torch.equal(out[:m], rows[:m]) and bool((out[m:] == SENTINEL).all()), m
            order = np.argsort(mi.cpu().numpy()[:len(want)])
            assert (mi.cpu().numpy()[:len(want)][order] == want).all() and (mk.cpu().numpy()[:len(want)][order] == keys[want]).all(), m
