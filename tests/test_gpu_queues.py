"""Walk groups are taken from eight queues: every group is walked exactly once
when queues are empty, hold one group, or run out while others are left."""
import numpy as np
import pytest

from paper_2609_17658_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def resident():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    n = 20000
    pos = torch.as_tensor(synth.mixture_box(n, 9), device="cuda")
    mass = torch.as_tensor(synth.equal_masses(n), device="cuda")
    prm = synth.scale_free_params(n).as_dict()
    trees = {g: og.Tree(pos, mass, 1.0, prm, stream=torch.cuda.current_stream(), group_max=g) for g in (1, 3, 64)}
    full = {p: trees[64].force(precision=p) for p in ("mixed", "fp64")}
    yield n, trees, full
    for t in trees.values():
        t.close()


# with one target per group: fewer groups than queues, one each, one more,
# several each and a ragged rest; and groups of 3 and 64
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("m,chunk", [(1, 1), (7, 1), (8, 1), (9, 1), (17, 1), (4099, 1), (25, 3), (20000, 64)])
def test_every_group_once(resident, m, chunk, precision):
    n, trees, full = resident
    print("queues m=%d chunk=%d %s" % (m, chunk, precision), flush=True)
    idx = torch.as_tensor(np.random.default_rng(m).permutation(n)[:m].copy(), device="cuda")
    acc = torch.full((m, 3), float("nan"), dtype=torch.float64, device="cuda")
    pot = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
    trees[chunk].force(targets=idx, precision=precision, acc=acc, pot=pot)
    assert torch.equal(acc, full[precision][0][idx]) and torch.equal(pot, full[precision][1][idx])
