"""The walk with eight lanes per target against the walks with one lane per
target (64 targets per wave), which it replaces for few targets: the terms and
their order are the same, so accelerations, potentials and interaction counts
must be the same to the bit, in both precisions.  OG_EIGHT_MAX sets up to how
many targets it is taken: 0 leaves every walk to the others, and in FP64 the
plain walk (OG_WALK64_PLAIN=1) is compared too.  Parity with the oracle comes
from the parity tests, whose small cases take this walk by default."""
import numpy as np
import pytest
from hypothesis import HealthCheck, given, settings

from paper_2609_17658_amd import synth
from prop_inputs import configs
from test_gpu_walk64_screen import CASES, _batch_items, _dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ALL = str(10 ** 9)


@pytest.fixture(scope="module")
def og_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    og.load()
    return og


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def _compare(og, monkeypatch, pos, mass, box, prm, targets=None, **kw):
    prm = dict(prm, **kw)
    eps = prm.pop("eps_lengths", None)
    if eps is not None:
        prm["eps_particle"] = _dev(eps)
    a_old = None
    if prm.get("criterion", 0) == 1:
        rng = np.random.default_rng(5)
        a_old = _dev(rng.standard_normal((pos.shape[0], 3)) * np.exp(rng.uniform(-3.0, 3.0, (pos.shape[0], 1))))
    tree = og.Tree(_dev(pos), _dev(mass), box, prm, stream=torch.cuda.current_stream())
    tg = None if targets is None else _dev(targets, torch.int64)

    def walk(precision, most, plain="0"):
        monkeypatch.setenv("OG_EIGHT_MAX", most)
        monkeypatch.setenv("OG_WALK64_PLAIN", plain)
        return [v.clone() for v in tree.force(targets=tg, precision=precision, with_counts=True, a_old=a_old)]

    for precision in ("mixed", "fp64"):
        eight = walk(precision, ALL)
        _same(eight, walk(precision, "0"))
        if precision == "fp64":
            _same(eight, walk(precision, "0", plain="1"))
    assert tree.status() == 0
    tree.close()


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_same_bits(og_mod, monkeypatch, case):
    name, pos, mass, box, prm = case
    print("eight lanes: %s N=%d" % (name, pos.shape[0]), flush=True)
    _compare(og_mod, monkeypatch, pos, mass, box, prm)


# ragged runs of eight and of 64, a leaf as root, big leaves, an opened
# everything (full queues), one-particle leaves (deep stacks), other groupings
@pytest.mark.parametrize("n,leaf_max,theta,group_max", [
    (1, 8, 0.5, 0), (7, 8, 0.5, 0), (8, 1, 0.5, 0), (9, 4, 0.0, 3), (63, 64, 0.5, 0), (65, 1, 0.0, 0),
    (513, 1, 0.3, 1), (1500, 200, 0.5, 0), (2049, 8, 0.0, 64)])
def test_edges(og_mod, monkeypatch, n, leaf_max, theta, group_max):
    print("eight lanes: n=%d leaf_max=%d theta=%g" % (n, leaf_max, theta), flush=True)
    rng = np.random.default_rng(n)
    pos = synth.wrap(np.concatenate([rng.random((n - n // 2, 3)), 0.7 + 0.003 * rng.standard_normal((n // 2, 3))]))
    prm = dict(G=1.0, eps=0.003, r_s=0.05, r_cut=0.225, theta=theta, periodic=1, leaf_max=leaf_max)
    _compare(og_mod, monkeypatch, pos, rng.uniform(0.5, 1.5, n) / n, 1.0, prm, group_max=group_max)


# r_cut up to nearly half the box (offsets of half a box have two images)
@pytest.mark.parametrize("r_cut", [0.2499, 0.2501, 0.4999])
def test_wide_cutoff(og_mod, monkeypatch, r_cut):
    rng = np.random.default_rng(8)
    pos = rng.random((3000, 3))
    pos[:200] = np.round(pos[:200] * 8) / 8 % 1.0
    prm = dict(G=1.0, eps=0.003, r_s=r_cut / 4.5, r_cut=r_cut, theta=0.5, periodic=1, leaf_max=4)
    _compare(og_mod, monkeypatch, pos, np.full(3000, 1 / 3000), 1.0, prm)


@pytest.mark.parametrize("m", [1, 5, 8, 4096])
def test_target_lists(og_mod, monkeypatch, m):
    name, pos, mass, box, prm = CASES[0]
    tg = np.random.default_rng(m).integers(0, pos.shape[0], m)  # with repeats
    print("eight lanes: %d targets" % m, flush=True)
    _compare(og_mod, monkeypatch, pos, mass, box, prm, targets=tg)


# active lists on both sides of the line (the choice is made on the device)
@pytest.mark.parametrize("line", [0, 2999, 3000, 10 ** 9])
def test_active_lists(og_mod, monkeypatch, line):
    name, pos, mass, box, prm = CASES[0]
    n = pos.shape[0]
    bins = torch.ones(n, dtype=torch.int8, device="cuda")
    bins[torch.randperm(n, generator=torch.Generator().manual_seed(4))[:3000].cuda()] = 0
    tree = og_mod.Tree(_dev(pos), _dev(mass), box, prm, stream=torch.cuda.current_stream())
    for precision in ("mixed", "fp64"):
        print("eight lanes: active, line %d, %s" % (line, precision), flush=True)
        monkeypatch.setenv("OG_EIGHT_MAX", "0")
        full, pot = tree.force(precision=precision)
        monkeypatch.setenv("OG_EIGHT_MAX", str(line))
        acc = torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda")
        ph = torch.full((n,), 7.0, dtype=torch.float64, device="cuda")
        count = torch.zeros(1, dtype=torch.int64, device="cuda")
        tree.force_active(bins, 0, acc, ph, precision=precision, n_active=count)
        on = bins == 0
        assert count.item() == 3000
        assert torch.equal(acc[on], full[on]) and torch.equal(ph[on], pot[on])
        assert bool((acc[~on] == 7.0).all()) and bool((ph[~on] == 7.0).all())
    tree.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batches(og_mod, monkeypatch, precision):
    items = _batch_items(True)
    got = []
    for most in ("0", ALL):
        monkeypatch.setenv("OG_EIGHT_MAX", most)
        b = og_mod.Batch(items, stream=torch.cuda.current_stream(), precision=precision, group_max=20)
        b.force()
        torch.cuda.synchronize()
        got.append([v.clone() for o in b.outputs for v in o])
        b.close()
    _same(*got)


@settings(max_examples=40, deadline=None, derandomize=True, database=None,
          suppress_health_check=[HealthCheck.too_slow, HealthCheck.data_too_large,
                                 HealthCheck.function_scoped_fixture])
@given(cfg=configs())
def test_generated_inputs(og_mod, monkeypatch, cfg):
    print("eight lanes: %s" % cfg.label, flush=True)
    _compare(og_mod, monkeypatch, cfg.pos, cfg.mass, cfg.box, cfg.params)
