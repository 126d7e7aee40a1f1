"""The build of a small box in one workgroup against the general build
(OG_NO_SMALL_BUILD=1): the exported tree, the forces and the status are the
same to the bit, and the tree passes the host-side check."""
import numpy as np
import pytest
from hypothesis import HealthCheck, given, settings

from prop_inputs import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


def _compare(og, monkeypatch, pos, mass, box, prm, check=True):
    tp = torch.as_tensor(np.ascontiguousarray(pos), device="cuda")
    tm = torch.as_tensor(np.ascontiguousarray(mass), device="cuda")
    got = []
    for off in ("0", "1"):
        monkeypatch.setenv("OG_NO_SMALL_BUILD", off)
        t = og.Tree(tp, tm, box, prm, stream=torch.cuda.current_stream())
        status = t.status()
        if check:
            assert status == 0
            t.validate()
        ex = t.export()
        stats = t.stats()
        f = [v.clone() for p in ("mixed", "fp64") for v in t.force(precision=p, with_counts=True)]
        monkeypatch.setenv("OG_EIGHT_MAX", "0")  # both forms of walk read the records
        f += [v.clone() for v in t.force(precision="mixed")]
        monkeypatch.delenv("OG_EIGHT_MAX")
        torch.cuda.synchronize()
        t.close()
        got.append((status, stats, ex, f))
    a, b = got
    assert a[0] == b[0] and a[1] == b[1]
    for k in a[2]:
        assert np.array_equal(a[2][k], b[2][k]), k
    for x, y in zip(a[3], b[3]):
        assert torch.equal(x, y)


# one particle to a full leaf and one more; odd counts around the wave and the
# workgroup; the largest box the node bound admits for the leaf size (1232 for
# 8, 357 for 1, 2048 for large leaves), and one particle more (general path)
@pytest.mark.parametrize("n,leaf_max", [(1, 8), (2, 1), (8, 8), (9, 8), (63, 4), (65, 16), (1000, 8), (1023, 8),
                                        (1025, 8), (1232, 8), (1233, 8), (357, 1), (358, 1), (2047, 64),
                                        (2048, 64), (2049, 64), (2048, 4096)])
@pytest.mark.parametrize("curve", ["morton", "hilbert"])
def test_same_tree(og_mod, monkeypatch, n, leaf_max, curve):
    print("small build n=%d leaf_max=%d %s" % (n, leaf_max, curve), flush=True)
    rng = np.random.default_rng(n + leaf_max)
    pos = rng.random((n, 3))
    pos[::2] = 0.6 + 0.01 * rng.standard_normal(pos[::2].shape)
    prm = dict(G=1.0, eps=0.004, r_s=0.05, r_cut=0.225, theta=0.5, periodic=1, leaf_max=leaf_max, curve=curve)
    _compare(og_mod, monkeypatch, pos, rng.uniform(0.5, 1.5, n) / n, 1.0, prm)


def test_deep_and_coincident(og_mod, monkeypatch):
    rng = np.random.default_rng(1)
    pos = rng.random((900, 3))
    pos[:300] = pos[0]                               # a leaf of 300 at the deepest level
    pos[300:600] = pos[300] + 2.0 ** -21 * rng.integers(0, 3, (300, 3))  # chains to the deepest level
    prm = dict(G=1.0, eps=0.004, r_s=0.05, r_cut=0.225, theta=0.5, periodic=1, leaf_max=8)
    _compare(og_mod, monkeypatch, pos % 1.0, np.full(900, 1 / 900), 1.0, prm)


@pytest.mark.parametrize("bad", [np.nan, -0.25, 1.0])
def test_status(og_mod, monkeypatch, bad):
    pos = np.random.default_rng(2).random((500, 3))
    pos[77, 1] = bad
    prm = dict(G=1.0, eps=0.004, r_s=0.05, r_cut=0.225, theta=0.5, periodic=1, leaf_max=8)
    for off in ("0", "1"):
        monkeypatch.setenv("OG_NO_SMALL_BUILD", off)
        t = og_mod.Tree(torch.as_tensor(pos, device="cuda"), torch.full((500,), 0.002, dtype=torch.float64, device="cuda"),
                        1.0, prm, stream=torch.cuda.current_stream())
        assert t.status() == og_mod.OG_ERANGE
        t.close()


@settings(max_examples=40, deadline=None, derandomize=True, database=None,
          suppress_health_check=[HealthCheck.too_slow, HealthCheck.data_too_large,
                                 HealthCheck.function_scoped_fixture])
@given(cfg=configs())
def test_generated_inputs(og_mod, monkeypatch, cfg):
    print("small build: %s" % cfg.label, flush=True)
    _compare(og_mod, monkeypatch, cfg.pos, cfg.mass, cfg.box, cfg.params)
