"""New gradient pointers at every step: tables of one launch, of several, and
of the staged copy (more than 512 tensors), in steps enqueued without waiting,
give the bits of the same gradients in fixed buffers."""
import pytest
import torch

from paper_2609_30342_amd import rikfad as R
from paper_2609_30342_amd import synth

from parity import log

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("count", [1, 255, 256, 257, 512, 513])
@pytest.mark.parametrize("kind", ["rikfad", "adafm"])
def test_new_pointers_every_step(kind, count):
    log(f"[case] {kind} gradient table of {count}")
    gen = torch.Generator(device="cuda").manual_seed(count)
    steps = 6
    shape = [(2 + i % 3, 4 + i % 5) for i in range(count)]
    x0 = [torch.randn(s, generator=gen, device="cuda") for s in shape]
    gs = [[torch.randn(s, generator=gen, device="cuda") for s in shape] for _ in range(steps)]

    def make(x, g):
        return R.RIKFAD(x, g, **synth.HP_FRICTION) if kind == "rikfad" else R.ADAFM(x, g, h=1e-2)

    xa, xb = [x.clone() for x in x0], [x.clone() for x in x0]
    buf = [g.clone() for g in gs[0]]
    a, b = make(xa, gs[0]), make(xb, buf)
    for s in range(steps):
        a.step(grads=gs[s])
    for s in range(steps):
        for d, g in zip(buf, gs[s]):
            d.copy_(g)
        b.step()
    torch.cuda.synchronize()
    assert all(torch.equal(p, q) for p, q in zip(xa, xb))
    a.close()
    b.close()
