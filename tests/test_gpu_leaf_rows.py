"""The mixed walk's evaluation of listed leaves, two particles at a time: leaves
of exactly c particles (odd and even, up to one list entry's 8 and past it),
around the periodic faces and inside, cut off and not, against the eight-lane
walk, which evaluates one item per lane (OG_EIGHT_MAX: up to how many targets it
is taken).  Terms and order are the same, so the results are the same to the
bit, at every list depth."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


def _clusters(c, rng):
    """c particles in each of 300 cells of a 16^3 grid, faces included."""
    cell = rng.permutation(16 ** 3)[:300]
    cell[:8] = [0, 15, 15 * 16, 15 * 256, 15 * 273, 255, 4095, 4080]
    at = np.stack([cell // 256, cell // 16 % 16, cell % 16], axis=1)[np.unique(cell, return_index=True)[1]]
    return ((at[:, None, :] + rng.random((len(at), c, 3))) / 16.0).reshape(-1, 3)


@pytest.mark.parametrize("kind", ["periodic", "open_cutoff", "newton"])
@pytest.mark.parametrize("c", [1, 2, 3, 7, 8, 9, 16, 17])
def test_leaves_of_c_particles(og_mod, monkeypatch, c, kind):
    rng = np.random.default_rng(c)
    pos = _clusters(c, rng)
    n = len(pos)
    cut = dict(r_s=0.0, r_cut=0.0) if kind == "newton" else dict(r_s=0.05, r_cut=0.2)
    prm = dict(G=1.0, eps=0.002, theta=0.4, periodic=int(kind == "periodic"), leaf_max=c, **cut)
    tp, tm = torch.as_tensor(pos, device="cuda"), torch.as_tensor(rng.uniform(0.5, 1.5, n) / n, device="cuda")
    ref = None
    for most, cap in (("1000000000", 0), ("0", 0), ("0", 4), ("0", 8)):
        print("leaves of %d, %s, eight-lane up to %s, depth %d" % (c, kind, most, cap), flush=True)
        monkeypatch.setenv("OG_EIGHT_MAX", most)
        t = og_mod.Tree(tp, tm, 1.0, dict(prm, walk_list_cap=cap), stream=torch.cuda.current_stream())
        got = [v.clone() for v in t.force(precision="mixed", with_counts=True)]
        assert t.status() == 0
        t.close()
        ref = ref or got
        for a, b in zip(ref, got):
            assert torch.equal(a, b)
    assert int(ref[2].sum()) > 0
