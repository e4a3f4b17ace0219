"""fstat_last_tile speaks of the last demodulation: a call that its band check
refuses has none, also where a launch was queued ahead of the check."""
import dataclasses

import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["compute", "noalloc"])
def test_a_refused_call_leaves_the_last_shape(tmp_path, entry):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(1800, n_det=1, slots=20, keep=1.0, n_sky=2, n_fd=4, n_f=200, injections=())
    wu, _ = to_device(w)
    cut = dataclasses.replace(wu, k_first=int(w.f0 * w.t_sft) + w.dterms)
    big = small_workload(1801, n_det=1, slots=6, keep=1.0, n_sky=60, n_fd=8, n_f=1536, injections=())
    out, big_out = alloc_output(w), alloc_output(big)
    with P.Plan(max_sft=w.n_sft, max_bins=big.n_bins, max_sky=60, max_fd=8, max_f=1536) as p:
        call = p.compute if entry == "compute" else p.compute_noalloc
        with pytest.raises(P.FstatError):
            call(cut, out)
        with pytest.raises(P.FstatError):          # no demodulation yet
            p.last_tile()
        p.compute(to_device(big)[0], big_out)
        before = p.last_tile()
        assert before["threads"] == 256
        with pytest.raises(P.FstatError):
            call(cut, out)
        assert p.last_tile() == before
        call(wu, out)
        torch.cuda.synchronize()
        assert p.last_tile()["threads"] == 64
