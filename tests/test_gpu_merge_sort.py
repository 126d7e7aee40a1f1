"""The merge sort that small boxes and short target lists take: the order is
the one of the keys with ties by caller index, as the oracle sorts them, at the
edges of tiles and of merges, and the same as the radix sort's
(OG_MERGE_MAX=0)."""
import numpy as np
import pytest

from paper_2609_17658_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


def _positions(n, seed):
    """A third uniform, a third on few distinct points (equal keys all over
    the list), a third in a cluster."""
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3))
    pos[::3] = rng.random((5, 3))[rng.integers(0, 5, len(pos[::3]))]
    pos[1::3] = 0.4 + 1e-4 * rng.standard_normal(pos[1::3].shape)
    return pos


# below four elements per thread, a full thread, one more; below, at and above
# a tile of 1024, a merge of eight (8192), two merges (65536), three (524288)
@pytest.mark.parametrize("curve", ["morton", "hilbert"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025, 2049, 8192, 8193, 65536, 65537, 530001])
def test_order(og_mod, oracle_mod, monkeypatch, n, curve):
    print("merge sort n=%d %s" % (n, curve), flush=True)
    monkeypatch.setenv("OG_MERGE_MAX", str(10 ** 9))
    pos = _positions(n, n)
    prm = dict(G=1.0, eps=0.01, r_s=0.02, r_cut=0.09, theta=0.5, periodic=1, leaf_max=8, curve=curve)
    t = og_mod.Tree(torch.as_tensor(pos, device="cuda"), torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda"),
                    1.0, prm, stream=torch.cuda.current_stream())
    got = t.export()
    assert t.status() == 0
    if n <= 70000:
        t.validate()
    t.close()
    keys = oracle_mod.keys(pos, 1.0, curve=1 if curve == "hilbert" else 0)
    perm = np.argsort(keys, kind="stable")
    assert np.array_equal(got["perm"], perm.astype(np.uint32))
    assert np.array_equal(got["keys"], keys[perm])


def test_batch_order(og_mod, monkeypatch):
    """Boxes of one tile, several and one particle, among them one with
    per-particle lengths and an open one."""
    items = []
    for b, n in enumerate([1, 1024, 700, 9000, 1025, 3, 70000]):
        prm = synth.scale_free_params(max(n, 1000)).as_dict()
        pos = torch.as_tensor(_positions(n, 90 + b), device="cuda")
        if b == 3:
            prm["eps_particle"] = torch.full((n,), 0.003, dtype=torch.float64, device="cuda")
        if b == 4:
            prm.update(periodic=0, r_s=0.0, r_cut=0.0)
        items.append((pos, torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda"), 1.0, prm))
    got = []
    for line in ("0", str(10 ** 9)):
        monkeypatch.setenv("OG_MERGE_MAX", line)
        b = og_mod.Batch(items, stream=torch.cuda.current_stream(), precision="fp64")
        b.force()
        torch.cuda.synchronize()
        assert b.status() == 0
        got.append([v.clone() for o in b.outputs for v in o])
        b.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("m", [1, 2, 1024, 1025, 16384, 16385])
def test_target_lists(og_mod, monkeypatch, m):
    n = 30000
    pos = torch.as_tensor(synth.mixture_box(n, 3), device="cuda")
    mass = torch.as_tensor(synth.equal_masses(n), device="cuda")
    t = og_mod.Tree(pos, mass, 1.0, synth.scale_free_params(n).as_dict(), stream=torch.cuda.current_stream())
    idx = torch.as_tensor(np.random.default_rng(m).integers(0, n, m), device="cuda")  # with repeats
    got = []
    for line in ("0", str(10 ** 9)):
        print("merge sort, %d targets, line %s" % (m, line), flush=True)
        monkeypatch.setenv("OG_MERGE_MAX", line)
        got.append([v.clone() for v in t.force(targets=idx, with_counts=True)])
    for x, y in zip(*got):
        assert torch.equal(x, y)
    assert t.status() == 0
    idx[m // 2] = n  # out of range: particle 0's result, reported
    acc, pot = t.force(targets=idx)
    full = t.force(targets=torch.zeros(1, dtype=torch.int64, device="cuda"))
    assert torch.equal(acc[m // 2], full[0][0]) and torch.equal(pot[m // 2], full[1][0])
    assert t.status() == og_mod.OG_ERANGE
    t.close()
