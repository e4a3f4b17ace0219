"""Interp tiles that keep a slot's coefficients for the next slot where no lane
of the wave moved to another bin: the arithmetic per template and SFT is that
of the kernel with one wave per template row, in the same order, so 2F, Fa and
Fb must equal its bit for bit, and the oracle's within its tolerance, whether
the spindown step moves the bins never, now and then, or at almost every slot
(past one bin per step the plain loop runs), for every block size of the
spindown split (chains of equal and of unequal length)."""
import numpy as np
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("shift", [0.0, 0.03, 0.5, 0.98, 1.5])
@pytest.mark.parametrize("n_fd", [4, 5, 6, 7, 8, 16, 21])
def test_shared_slots_equal_the_wave_kernel(torch_cuda, oracle_lib, tmp_path, n_fd, shift):
    import paper_0904_1826_amd as P
    torch = torch_cuda
    kw = dict(n_det=1, slots=21, keep=1.0, n_sky=3, n_fd=n_fd, n_f=330, injections=((1, n_fd - 1, 200, 12.0),))
    w = small_workload(990, **kw)
    tau = (w.t_start + 0.5 * w.t_sft - w.t_ref)[None, :] + w.sky @ w.pos.T
    step = shift / (float(np.abs(tau).max()) * w.t_sft)              # spindown step that moves the bins by `shift`
    w = small_workload(990, fdot_lo=-step * (n_fd - 1), **kw)
    wu, _ = to_device(w)
    cache = tmp_path / "tiles.txt"
    cache.write_text("s0_d8_k0_c0 8 4 0 256\n")
    outs = []
    for tiles in (False, True):
        o = alloc_output(w, fafb=True)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=w.n_sky, max_fd=n_fd, max_f=w.n_f) as p:
            if tiles:
                p.autotune(wu, o, cache_path=str(cache))
            p.compute(wu, o)
            torch.cuda.synchronize()
            if tiles:
                assert p.last_tile()["nf_reg"] == 8
        outs.append(o)
    for name in ("twoF", "fa", "fb"):
        assert torch.equal(getattr(outs[0], name), getattr(outs[1], name)), name
    e = twoF_error(outs[1].twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"])
    assert e.max() <= 1e-4
