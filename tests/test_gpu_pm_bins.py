"""The mesh force of caller-order particles deposited by blocks (numbers sorted
by block first) against the per-particle deposit: the fixed-point sums do not
depend on the order, so the results are the same to the bit.
OG_PM_BIN_MIN=n sets from how many particles the blocks are taken."""
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


# one block whose halo wraps onto itself; small and larger meshes; one
# particle; more particles than the scratch in the mesh holds (falls back);
# blocks of more than 2048 particles (the rest taken one by one)
@pytest.mark.parametrize("n_grid,n,clump", [(8, 200, 0.0), (16, 1500, 0.0), (32, 1, 0.0), (32, 40000, 0.0),
                                            (64, 60001, 0.5), (128, 300000, 0.7)])
def test_same_bits(og_mod, monkeypatch, n_grid, n, clump):
    print("mesh blocks n_grid=%d n=%d" % (n_grid, n), flush=True)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)) * 3.0
    k = int(clump * n)
    pos[:k] = 1.1 + 0.01 * rng.standard_normal((k, 3))
    m = min(n, 40)
    pos[:m] = np.where(rng.random((m, 3)) < 0.5, 0.0, np.nextafter(3.0, 0.0))  # on the periodic faces
    pos[n // 2:n // 2 + m] += rng.integers(-2, 3, (len(pos[n // 2:n // 2 + m]), 3)) * 3.0  # outside: wrapped
    pos = pos[rng.permutation(n)]
    tp = torch.as_tensor(pos, device="cuda")
    tm = torch.as_tensor(rng.uniform(0.5, 1.5, n) / n, device="cuda")
    mesh = og_mod.PM(n_grid, 3.0, 1.3, 3.75 / n_grid, stream=torch.cuda.current_stream())
    got = []
    for line in (str(2 ** 31), "0"):
        monkeypatch.setenv("OG_PM_BIN_MIN", line)
        for rep in range(2):
            got.append([v.clone() for v in mesh.force(tp, tm)])
    mesh.close()
    for g in got[1:]:
        assert torch.equal(g[0], got[0][0]) and torch.equal(g[1], got[0][1])
