"""Tiles of two sky points in each form of their slots (plain, shared, shared
with the words read), for every block size that pairs: the form is the one
asked for, the tiles are paired, and 2F, Fa and Fb equal those of tiles that
neither pair nor share, bit for bit; alone and in a batch.  The sky points are
a patch dense enough to pair at the highest of the frequencies."""
import numpy as np
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import replace, small_workload, twoF_error

pytestmark = pytest.mark.gpu

N_SKY = 21


def _patch(w):
    """The unit with its sky points moved into a patch of 0.05 rad."""
    i = np.arange(N_SKY)
    n = np.array([0.6, 0.5, 0.62]) + 0.01 * np.stack([i % 5, i // 5, 0 * i], 1)
    return replace(w, sky=n / np.linalg.norm(n, axis=1, keepdims=True))


@pytest.mark.parametrize("f0,shift,form", [(431.0, 0.5, 1), (800.0, 0.5, 2), (800.0, 0.98, 2), (800.0, 1.5, 0)])
@pytest.mark.parametrize("n_fd", [4, 5, 6, 7, 8])
def test_paired_tiles_in_every_form(oracle_lib, tmp_path, n_fd, f0, shift, form):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    kw = dict(n_det=1, slots=21, keep=1.0, n_sky=N_SKY, n_fd=n_fd, n_f=330, f0=f0, injections=())
    w = _patch(small_workload(1600, fdot_lo=-1e-9, **kw))
    tau = (w.t_start + 0.5 * w.t_sft - w.t_ref)[None, :] + w.sky @ w.pos.T
    max_tau = float(np.abs(tau).max())
    step = shift / (max_tau * w.t_sft)
    w = _patch(small_workload(1600, fdot_lo=-step * (n_fd - 1), **kw))
    assert P.fstat_slot_form([(w.df, w.dfdot, w.t_sft, w.k_first, w.n_bins, max_tau, 1)]) == form
    wu, _ = to_device(w)
    outs = []
    for waves in (4, 3, 0):                               # 0: the batched form
        cache = tmp_path / f"tiles{waves}.txt"
        cache.write_text(f"s0_d8_k0_c0 8 {waves or 4} 0 256\nbatch_s0_c0 8 256 256 256\n")
        o = alloc_output(w, fafb=True)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=N_SKY, max_fd=n_fd, max_f=w.n_f) as p:
            p.autotune(wu, o, cache_path=str(cache))
            if waves:
                p.compute(wu, o)
            else:
                p.batch_compute([wu], [o])
            torch.cuda.synchronize()
            if waves:
                assert (p.last_tile()["pair_seg"] > 0) == (waves == 4), p.last_tile()
        outs.append(o)
    for o in outs[1:]:
        for name in ("twoF", "fa", "fb"):
            assert torch.equal(getattr(outs[0], name), getattr(o, name)), name
    assert twoF_error(outs[0].twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"]).max() <= 1e-4


def test_choice_of_pairs_does_not_change_a_unit_that_fills_the_device(tmp_path):
    """256 x 8 x 3071 runs paired by the rule; three waves per SIMD never pair."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(1010, n_det=1, slots=6, keep=1.0, n_sky=256, n_fd=8, n_f=3071, f0=60.0, injections=())
    wu, _ = to_device(w)
    cache = tmp_path / "tiles.txt"
    cache.write_text("s0_d8_k0_c0 8 3 0 256\nbatch_s0_c0 8 256 256 256\n")
    outs = []
    for tuned in (False, True):
        o = alloc_output(w)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=256, max_fd=8, max_f=3071) as p:
            if tuned:
                p.autotune(wu, o, cache_path=str(cache))
            p.compute(wu, o)
            torch.cuda.synchronize()
            assert (p.last_tile()["pair_seg"] > 0) != tuned, p.last_tile()
        outs.append(o)
    assert torch.equal(outs[0].twoF, outs[1].twoF)
