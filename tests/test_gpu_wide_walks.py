"""The 64-target walks by themselves (OG_EIGHT_MAX=0: the small inputs of the
other tests take the walk with eight lanes per target), and the group queues
while waves take more than one group: group sizes, list depths, interior groups
and record offsets do not change a bit, the results agree with the oracle, and
every group is walked exactly once."""
import numpy as np
import pytest

from paper_2609_17658_amd import synth
from test_gpu_parity import CASES, gpu_run, oracle_params, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ALL = str(10 ** 9)
NAMES = [c[0] for c in CASES]


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


@pytest.fixture(autouse=True)
def wide(monkeypatch):
    monkeypatch.setenv("OG_EIGHT_MAX", "0")


def _same(a, b, what):
    for k in ("acc", "pot", "nint"):
        assert np.array_equal(a[k], b[k]), (k, what)


@pytest.mark.parametrize("name", NAMES)
def test_oracle(og_mod, oracle_mod, name):
    _, pos, mass, box, prm = CASES[NAMES.index(name)]
    acc, pot, nint = oracle_mod.tree_force(pos, mass, box, oracle_params(oracle_mod, prm))
    ok = np.linalg.norm(acc, axis=1) > 0
    for plain in ("0", "1"):
        with pytest.MonkeyPatch.context() as m:
            m.setenv("OG_WALK64_PLAIN", plain)
            print("wide walks, oracle: %s fp64 plain=%s" % (name, plain), flush=True)
            g = gpu_run(og_mod, pos, mass, box, prm, precision="fp64")
        assert g["status"] == 0 and np.array_equal(g["nint"], nint)
        assert rel_err(g["acc"], acc).max() <= 1e-11
        assert np.all(np.abs(g["pot"] - pot) <= 1e-12 * np.abs(pot) + 1e-300)
    g = gpu_run(og_mod, pos, mass, box, prm, precision="mixed")
    if ok.any():
        e = rel_err(g["acc"], acc)[ok]
        assert np.median(e) <= 1e-3 and np.percentile(e, 99) <= 1e-2
        assert (g["nint"] != nint).mean() <= 0.01


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", ["mixture32k", "rand10007_lm16", "box3_faces", "open3000"])
def test_group_sizes(og_mod, name, precision):
    _, pos, mass, box, prm = CASES[NAMES.index(name)]
    ref = gpu_run(og_mod, pos, mass, box, prm, precision=precision)
    for gm in (64, 32, 7, 1):
        print("wide walks, groups of %d: %s %s" % (gm, name, precision), flush=True)
        _same(gpu_run(og_mod, pos, mass, box, prm, precision=precision, group_max=gm), ref, gm)


@pytest.mark.parametrize("variant", [{}, {"softening": "spline"}, {"curve": "hilbert"}])
@pytest.mark.parametrize("name", ["mixture32k", "rand10007_lm16", "coincident300", "box3_faces", "open3000",
                                  "open_cut4000"])
def test_list_depths(og_mod, name, variant):
    _, pos, mass, box, prm = CASES[NAMES.index(name)]
    ref = gpu_run(og_mod, pos, mass, box, prm, precision="mixed", **variant)
    for cap in (4, 8, 16, 32):
        print("wide walks, lists of %d: %s %s" % (cap, name, variant), flush=True)
        _same(gpu_run(og_mod, pos, mass, box, prm, precision="mixed", walk_list_cap=cap, **variant), ref, cap)


@pytest.mark.parametrize("switch", ["OG_NO_INTERIOR", "OG_WIDE_NODES"])
@pytest.mark.parametrize("name", ["mixture32k", "rand10007_lm16", "coincident300", "box3_faces", "rcut8rs5000"])
def test_other_forms(og_mod, monkeypatch, name, switch):
    _, pos, mass, box, prm = CASES[NAMES.index(name)]
    ref = gpu_run(og_mod, pos, mass, box, prm, precision="mixed")
    monkeypatch.setenv(switch, "1")
    print("wide walks, %s: %s" % (switch, name), flush=True)
    _same(gpu_run(og_mod, pos, mass, box, prm, precision="mixed"), ref, switch)


@pytest.fixture(scope="module")
def resident(og_mod):
    n = 50000
    pos = torch.as_tensor(synth.mixture_box(n, 9), device="cuda")
    mass = torch.as_tensor(synth.equal_masses(n), device="cuda")
    prm = synth.scale_free_params(n).as_dict()
    trees = {g: og_mod.Tree(pos, mass, 1.0, prm, stream=torch.cuda.current_stream(), group_max=g) for g in (1, 3, 64)}
    with pytest.MonkeyPatch.context() as m:
        m.setenv("OG_EIGHT_MAX", "0")
        full = {p: trees[64].force(precision=p) for p in ("mixed", "fp64")}
    yield n, trees, full
    for t in trees.values():
        t.close()


# With one target per group: fewer groups than queues, one each, one more,
# several each and a ragged rest; more groups than the launch has waves (8192 of
# the mixed walk, 7168 of the screened and 4096 of the plain FP64 walk), so that
# waves come back to their range and move on to others; groups of 3 and 64.  With
# eight lanes, more than 8 x 18 (FP64: 20) waves per compute unit's targets.
@pytest.mark.parametrize("walk", ["mixed", "fp64", "fp64 plain", "mixed eight", "fp64 eight"])
@pytest.mark.parametrize("m,chunk", [(1, 1), (7, 1), (8, 1), (9, 1), (17, 1), (4099, 1), (20011, 1), (50000, 1), (25, 3),
                                     (49999, 3), (20000, 64)])
def test_every_group_once(resident, monkeypatch, m, chunk, walk):
    n, trees, full = resident
    precision = walk.split()[0]
    monkeypatch.setenv("OG_EIGHT_MAX", ALL if "eight" in walk else "0")
    monkeypatch.setenv("OG_WALK64_PLAIN", "1" if "plain" in walk else "0")
    print("queues m=%d chunk=%d %s" % (m, chunk, walk), flush=True)
    idx = torch.as_tensor(np.random.default_rng(m).permutation(n)[:m].copy(), device="cuda")
    acc = torch.full((m, 3), float("nan"), dtype=torch.float64, device="cuda")
    pot = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
    trees[chunk].force(targets=idx, precision=precision, acc=acc, pot=pot)
    assert torch.equal(acc, full[precision][0][idx]) and torch.equal(pot, full[precision][1][idx])


@pytest.mark.parametrize("walk", ["mixed", "fp64", "mixed eight", "fp64 eight"])
@pytest.mark.parametrize("chunk", [1, 64])
def test_whole_box(resident, monkeypatch, chunk, walk):
    """All particles of the box: 50000 groups of one, or of 64."""
    n, trees, full = resident
    precision = walk.split()[0]
    monkeypatch.setenv("OG_EIGHT_MAX", ALL if "eight" in walk else "0")
    print("queues, whole box, chunk=%d %s" % (chunk, walk), flush=True)
    acc, pot = trees[chunk].force(precision=precision)
    assert torch.equal(acc, full[precision][0]) and torch.equal(pot, full[precision][1])


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025])
@pytest.mark.parametrize("curve", ["morton", "hilbert"])
def test_general_build_of_small_boxes(og_mod, oracle_mod, monkeypatch, n, curve):
    """The merge sort below and at one tile, the radix sort and the build in one
    workgroup: the oracle's order, and the same tree to the bit."""
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3))
    pos[::3] = rng.random((5, 3))[rng.integers(0, 5, len(pos[::3]))]
    prm = dict(G=1.0, eps=0.01, r_s=0.02, r_cut=0.09, theta=0.5, periodic=1, leaf_max=8, curve=curve)
    tp, tm = torch.as_tensor(pos, device="cuda"), torch.as_tensor(rng.uniform(0.5, 1.5, n) / n, device="cuda")
    keys = oracle_mod.keys(pos, 1.0, curve=1 if curve == "hilbert" else 0)
    perm = np.argsort(keys, kind="stable")
    ref = None
    for small, line in (("0", ALL), ("1", ALL), ("1", "0")):
        print("build n=%d %s general=%s merge line %s" % (n, curve, small, line), flush=True)
        monkeypatch.setenv("OG_NO_SMALL_BUILD", small)
        monkeypatch.setenv("OG_MERGE_MAX", line)
        t = og_mod.Tree(tp, tm, 1.0, prm, stream=torch.cuda.current_stream())
        got = t.export()
        assert t.status() == 0
        t.validate()
        force = [v.clone() for v in t.force(precision="fp64")]
        t.close()
        assert np.array_equal(got["perm"], perm.astype(np.uint32)) and np.array_equal(got["keys"], keys[perm])
        ref = ref or (got, force)
        for k in got:
            assert np.array_equal(got[k], ref[0][k]), (k, small, line)
        for a, b in zip(force, ref[1]):
            assert torch.equal(a, b)
