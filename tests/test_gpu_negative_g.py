"""A negative G (repulsion) in the mixed walks: a list entry's kind is told by the
sign of G m in the 64-target walk, which therefore does not take such boxes.
Terms and decisions (of the geometric criterion) do not depend on the sign, so
the results are those of +G with the sign turned, to the bit."""
import numpy as np
import pytest

from paper_2609_17658_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# below and above the line between the walks; with it at 0
@pytest.mark.parametrize("n,line", [(3000, None), (3000, "0"), (200001, None)])
@pytest.mark.parametrize("lists", ["target", "group"])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_turned_sign(monkeypatch, n, line, lists, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17658_amd import og
    if line is not None:
        monkeypatch.setenv("OG_EIGHT_MAX", line)
    print("negative G: n=%d line %s %s %s" % (n, line, lists, precision), flush=True)
    pos = torch.as_tensor(synth.mixture_box(n, 5), device="cuda")
    mass = torch.as_tensor(np.random.default_rng(5).uniform(0.5, 1.5, n) / n, device="cuda")
    idx = torch.arange(0, n, 7, device="cuda")
    bins = (torch.arange(n, device="cuda") % 5).to(torch.int8)
    got = []
    for g in (1.5, -1.5):
        prm = dict(synth.scale_free_params(n).as_dict(), G=g, lists=lists)
        t = og.Tree(pos, mass, 1.0, prm, stream=torch.cuda.current_stream())
        out = [*t.force(precision=precision, with_counts=True)]
        out += [*t.force(targets=idx, precision=precision)]
        acc = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
        pot = torch.zeros(n, dtype=torch.float64, device="cuda")
        t.force_active(bins, 1, acc, pot, precision=precision)
        torch.cuda.synchronize()
        assert t.status() == 0
        t.validate()
        t.close()
        got.append(out + [acc, pot])
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b if k == 2 else -b), k
