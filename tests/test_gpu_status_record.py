"""A geometry pass that finds its status record in a state that an earlier pass
did not leave clear (forced from the host: an arrival count that no pass can
complete) publishes nothing: the call says so instead of reading the result of
the call before it, a demodulation queued ahead of the check writes nothing
although the gate still stands from that call, and the next call is whole
again."""
import dataclasses

import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["interp", "direct"])
@pytest.mark.parametrize("entry,n_sky", [("compute", 2), ("compute", 6), ("noalloc", 2)])
def test_spoilt_record_is_an_error_and_heals(oracle_lib, monkeypatch, entry, n_sky, kernel):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    monkeypatch.setenv("FSTAT_FAULT", "record:2")
    w = small_workload(1300, n_det=2, slots=20, keep=1.0, n_sky=n_sky, n_fd=4, n_f=200,
                       injections=((1, 2, 90, 12.0),))
    wu, _ = to_device(w)
    cut = dataclasses.replace(wu, k_first=int(w.f0 * w.t_sft) + w.dterms)       # would fail its band check
    out = alloc_output(w)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=4, max_f=200, kernel=kernel) as p:
        call = p.compute if entry == "compute" else p.compute_noalloc
        call(wu, out)
        torch.cuda.synchronize()
        out.twoF.fill_(-1.0)
        with pytest.raises(P.FstatError) as e:
            call(cut, out)
        assert e.value.code == P.FSTAT_E_DEVICE and "no result" in p.last_error()
        torch.cuda.synchronize()
        assert bool((out.twoF == -1.0).all())
        with pytest.raises(P.FstatError) as e:
            call(cut, out)
        assert e.value.code == P.FSTAT_E_BAND
        call(wu, out)
        torch.cuda.synchronize()
    assert twoF_error(out.twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"]).max() <= 1e-4
