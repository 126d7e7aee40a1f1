"""Node ranks and active lists by the one-launch scan, at the edges of its tiles
(4096 values) and past the largest grid (2048 runs of tiles): the trees pass the
host-side check, alone and in a batch, and an active list equals the target
list of the same particles to the bit, with the exact count."""
import numpy as np
import pytest

from paper_2609_17658_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = 4096


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


def _box(n, seed):
    g = torch.Generator().manual_seed(seed)
    pos = torch.rand((n, 3), generator=g, dtype=torch.float64).cuda()
    return pos, torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda"), synth.scale_free_params(n).as_dict()


def _active_equals_targets(og, t, n, every):
    bins = torch.ones(n, dtype=torch.int8, device="cuda")
    bins[::every] = 0
    acc = torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda")
    na = torch.zeros(1, dtype=torch.int64, device="cuda")
    t.force_active(bins, 0, acc, n_active=na)
    idx = torch.nonzero(bins == 0).flatten()
    assert int(na) == len(idx)
    assert torch.equal(acc[idx], t.force(targets=idx, precision="mixed")[0])
    assert bool((acc[bins == 1] == 7.0).all())


@pytest.mark.parametrize("n", [1300, TILE - 1, TILE, TILE + 1, 3 * TILE, 3 * TILE + 5])
def test_tile_edges(og_mod, n):
    print("scan: n=%d" % n, flush=True)
    pos, mass, prm = _box(n, n)
    t = og_mod.Tree(pos, mass, 1.0, prm, stream=torch.cuda.current_stream())
    assert t.status() == 0
    t.validate()
    for every in (1, 3, n):
        _active_equals_targets(og_mod, t, n, every)
    t.close()
    items = [(pos, mass, 1.0, prm), _box(TILE + 7, 2)[:2] + (1.0, synth.scale_free_params(TILE + 7).as_dict())]
    b = og_mod.Batch(items, stream=torch.cuda.current_stream())
    outs = [a.clone() for a, _ in b.force()]
    assert b.status() == 0
    b.close()
    for (p, m, box, q), acc in zip(items, outs):
        t = og_mod.Tree(p, m, box, q, stream=torch.cuda.current_stream())
        assert torch.equal(acc, t.force(precision="mixed")[0])
        t.close()


def test_runs_of_tiles(og_mod):
    n = 2049 * TILE + 1
    print("scan: n=%d" % n, flush=True)
    pos, mass, prm = _box(n, 1)
    t = og_mod.Tree(pos, mass, 1.0, prm, stream=torch.cuda.current_stream())
    assert t.status() == 0
    _active_equals_targets(og_mod, t, n, 100003)
    t.validate()
    full = t.force(precision="mixed")[0]
    idx = torch.arange(0, n, 100003, device="cuda")
    assert torch.equal(full[idx], t.force(targets=idx, precision="mixed")[0])
    t.close()
