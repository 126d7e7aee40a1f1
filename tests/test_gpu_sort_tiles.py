"""The radix sort in tiles of 1024 keys, which the mesh deposit by blocks takes up
to 1.2 million particles, and in tiles of 4096 past it: the deposit by blocks
equals the one by atomics to the bit on both sides, at full and ragged tiles."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_grid,n", [(16, 1), (32, 1023), (32, 1024), (32, 1025), (64, 4097), (64, 60001),
                                      (128, 500000), (128, 1200000), (128, 1200001)])
def test_same_bits(monkeypatch, n_grid, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    print("sort tiles n_grid=%d n=%d" % (n_grid, n), flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    pos = torch.rand((n, 3), generator=g, dtype=torch.float64, device="cuda")
    pos[::2] = (0.3 + 0.05 * torch.randn(pos[::2].shape, generator=g, dtype=torch.float64, device="cuda")) % 1.0
    mass = (0.5 + torch.rand(n, generator=g, dtype=torch.float64, device="cuda")) / n
    mesh = og.PM(n_grid, 1.0, 1.0, 1.25 / n_grid, stream=torch.cuda.current_stream())
    got = []
    for line in (str(2 ** 31 - 1), "0"):
        monkeypatch.setenv("OG_PM_BIN_MIN", line)
        got.append([v.clone() for v in mesh.force(pos, mass)])
    mesh.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
