"""Adafactor-m sets whose update pass folds the tile sums of U^2 and X^2 itself
against the same steps with a separate scale launch (timed steps make one):
the same bits, for tensors of one tile to 64 and 256 tiles and one set beyond
the fold's range; and sets whose gradients the RMS pass keeps cached, against
the oracle through the update pass that reads them in reverse."""
import pytest
import torch

from paper_2609_30342_amd import rikfad as R
from paper_2609_30342_amd import synth

from parity import assert_ok, log, run_adafm_parity

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

S = synth.TensorSpec


@pytest.mark.parametrize("scale", [False, True])
@pytest.mark.parametrize("shapes", [
    [(3, 5), (1, 7), (40, 256), (2048, 256), (2080, 256), (1, 8192 * 3)],
    [(8192, 256), (8190, 255), (1, 2)],                      # 256 tiles of 32 rows
    [(8224, 256), (64, 64)],                                 # 257: beyond the fold
    [(8, 8)] * 2048, [(8, 8)] * 2049,        # tiles of a few elements: folded up to 2,048
], ids=["small", "256_tiles", "257_tiles", "2048_small_tiles", "2049_small_tiles"])
def test_folded_scale_has_the_same_bits(shapes, scale):
    log(f"[case] adafm folded scale {shapes} scale_parameter={scale}")
    got = []
    for timed in (False, True):
        gen = torch.Generator(device="cuda").manual_seed(4)
        xs = [torch.randn(s, generator=gen, device="cuda") for s in shapes]
        gs = [torch.randn(s, generator=gen, device="cuda") * 3 for s in shapes]
        opt = R.ADAFM(xs, gs, h=1e-2, scale_parameter=scale, clip_threshold=0.5)
        R.adafm_timing_enable(opt.ctx, timed)
        for _ in range(3):
            opt.step()
        torch.cuda.synchronize()
        got.append(xs + [t for st in opt.state for t in st])
        opt.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("specs", [
    [S("a", 3000, 768), S("b", 1, 768), S("c", 700, 1000, "bf16"), S("d", 90, 27),
     S("e", 40, 3, "bf16"), S("f", 1, 50, "bf16")],
    [S(f"t{i}", 5, 8) for i in range(7)], [S(f"t{i}", 5, 8) for i in range(8)],
    [S(f"t{i}", 5, 8) for i in range(17)],       # below, at and past whole eights of tiles
], ids=["mixed_types", "7_tiles", "8_tiles", "17_tiles"])
@pytest.mark.parametrize("clip", [1.0, 0.0])     # without clipping in launch order
def test_update_in_reverse_over_several_launches(specs, clip):
    log(f"[case] adafm reverse update {specs} clip={clip}")
    _, errs = run_adafm_parity(specs, dict(h=1e-2, scale_parameter=True, clip_threshold=clip), 4,
                               seed=9, label="reverse update")
    assert_ok(errs, label="reverse update")
