"""A call whose band check fails leaves nothing under way on its stream: its
coefficient passes (0.2 to 2 ms here, queued ahead of the check) are over when it
returns, so that the next call on the plan, on another stream, has the plan's
scratch and tables to itself and gives the oracle's values."""
import dataclasses

import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu


def _failing(n_sky, n_bins, n_sft):
    """A unit of pure noise whose first frequency lies below the band."""
    import torch
    w = small_workload(1200, n_det=1, slots=n_sft, keep=1.0, n_sky=n_sky, n_fd=3, n_f=150, dterms=16, noise=False,
                       injections=())
    wu, _ = to_device(w)
    sft = torch.randn((w.n_sft, n_bins, 2), device="cuda")
    return w, dataclasses.replace(wu, sft=sft, k_first=int(w.f0 * w.t_sft) + w.dterms)


@pytest.mark.parametrize("entry,n_sky", [("compute", 2), ("compute", 6), ("noalloc", 2), ("batch", 2), ("batch", 6),
                                         ("semicoherent", 6)])
def test_nothing_is_under_way_after_a_failed_check(oracle_lib, entry, n_sky):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    bw, bad = _failing(n_sky, 6000, 300 if entry == "noalloc" else 1500)
    good = small_workload(1201, n_det=2, slots=40, keep=1.0, n_sky=n_sky, n_fd=3, n_f=150, dterms=16,
                          injections=((1, 1, 90, 12.0),))
    wu, _ = to_device(good)
    out, spare = alloc_output(good), alloc_output(bw)
    second = {id(out): alloc_output(good), id(spare): alloc_output(bw)}
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    calls = {"compute": lambda p, u, o, s: p.compute(u, o, stream=s),
             "noalloc": lambda p, u, o, s: p.compute_noalloc(u, o, stream=s),
             "batch": lambda p, u, o, s: p.batch_compute([u, u], [o, second[id(o)]], stream=s),
             "semicoherent": lambda p, u, o, s: p.semicoherent([u], o, stream=s)}
    with P.Plan(max_sft=bad.n_sft, max_bins=6000, max_sky=n_sky, max_fd=3, max_f=150) as p:
        call = calls[entry]
        call(p, wu, out, b)                        # buffers and tables in place
        torch.cuda.synchronize()
        out.twoF.fill_(-1.0)
        torch.cuda.synchronize()
        for _ in range(2):
            with pytest.raises(P.FstatError) as e:
                call(p, bad, spare, a)
            assert e.value.code == P.FSTAT_E_BAND
            assert a.query(), "work of the failed call is still under way"
            call(p, wu, out, b)
        torch.cuda.synchronize()
    e = twoF_error(out.twoF.cpu().numpy().ravel(), oracle_lib.fstat(good)["twoF"])
    assert e.max() <= 1e-4, e.max()
