"""Units of one or two spindowns on both sides of the lines between one wave
per template row and tiles (templates, SFTs times how far the step exceeds
half a bin, spindowns, coefficient form): the form that the rule names runs,
and gives bit for bit what the tile gives."""
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload

pytestmark = pytest.mark.gpu


# the step is one bin
@pytest.mark.parametrize("n_sft,n_sky,n_fd,n_f,coef,wave", [
    (300, 200, 1, 2048, "f32", True), (302, 200, 1, 2048, "f32", False), (302, 190, 1, 2048, "f32", True),
    (40, 73, 2, 2048, "f32", True), (40, 74, 2, 2048, "f32", False),
    (600, 200, 1, 2048, "f16", True), (602, 200, 1, 2048, "f16", False), (602, 90, 2, 2048, "f16", True),
    (602, 100, 2, 2048, "f16", False)])
def test_one_or_two_spindowns(tmp_path, n_sft, n_sky, n_fd, n_f, coef, wave):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(1400, n_det=1, slots=n_sft, keep=1.0, n_sky=n_sky, n_fd=n_fd, n_f=n_f,
                       fdot_lo=-1e-12 if n_fd > 1 else 0.0, injections=())
    wu, _ = to_device(w)
    cache = tmp_path / "tiles.txt"
    cache.write_text(f"s0_d8_k0_c{int(coef == 'f16')} {n_fd} 3 0 256\nbatch_s0_c{int(coef == 'f16')} 8 256 256 256\n")
    outs = []
    for tuned in (False, True):
        o = alloc_output(w)
        with P.Plan(max_sft=n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=n_fd, max_f=n_f, coef=coef) as p:
            if tuned:
                p.autotune(wu, o, cache_path=str(cache))
            p.compute(wu, o)
            torch.cuda.synchronize()
            assert (p.last_tile()["threads"] == 64) == (wave and not tuned), p.last_tile()
        outs.append(o)
    assert torch.equal(outs[0].twoF, outs[1].twoF)
