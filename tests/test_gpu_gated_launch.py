"""The wave kernel queued before the host has seen the check (units of up to
three sky points or on the static scratch, without a toplist), gated on the
device: a check that fails leaves every output as it was, and one that passes
with a block of 16 spindowns outgrowing the slice leaves the unit to the tiles."""
import dataclasses

import numpy as np
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("coef,phase", [("f32", "fp64"), ("f16", "split")])
@pytest.mark.parametrize("entry,n_sky", [("compute", 1), ("compute", 3), ("noalloc", 3), ("noalloc", 7)])
def test_failed_checks_leave_the_outputs(oracle_lib, entry, n_sky, coef, phase):
    torch = _torch()
    import paper_0904_1826_amd as P
    w = small_workload(1500, n_det=2, slots=40, keep=1.0, n_sky=n_sky, n_fd=5, n_f=333, injections=((0, 2, 90, 12.0),))
    wu, _ = to_device(w)
    k, _, _, _ = oracle_lib.bins(w, oracle_lib.all_templates(w))
    first = int(k.min()) - w.dterms + 1 - w.k_first                # first column that a window reads
    short = dataclasses.replace(wu, sft=wu.sft[:, first + 1:].contiguous(), k_first=w.k_first + first + 1)
    singular = dataclasses.replace(wu, b=wu.a.clone())
    out = alloc_output(w, fafb=True)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=5, max_f=333, coef=coef, phase=phase) as p:
        call = p.compute if entry == "compute" else p.compute_noalloc
        for unit, code in ((short, P.FSTAT_E_BAND), (singular, P.FSTAT_E_ARG), (short, P.FSTAT_E_BAND)):
            for x in (out.twoF, out.fa, out.fb):
                x.fill_(-7.0)
            with pytest.raises(P.FstatError) as e:
                call(unit, out)
            torch.cuda.synchronize()
            assert e.value.code == code
            assert all(bool((x == -7.0).all()) for x in (out.twoF, out.fa, out.fb))
            assert p.last_kernel_ms() < 0
            call(wu, out)
            torch.cuda.synchronize()
            assert p.last_tile()["threads"] == 64
            e = twoF_error(out.twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"])
            assert e.max() <= (5e-3 if coef == "f16" else 1e-4)


@pytest.mark.parametrize("entry,n_sky", [("compute", 2), ("noalloc", 6)])
def test_gate_closed_by_the_slice_alone(oracle_lib, entry, n_sky):
    torch = _torch()
    import paper_0904_1826_amd as P
    kw = dict(n_det=2, slots=40, keep=1.0, n_sky=n_sky, n_fd=3, n_f=333, injections=((0, 1, 90, 12.0),))
    w = small_workload(1510, **kw)
    tau = (w.t_start + 0.5 * w.t_sft - w.t_ref)[None, :] + w.sky @ w.pos.T
    step = 50.0 / (15 * float(np.abs(tau).max()) * w.t_sft)       # 16 spindowns move the bins by 50, 4 by 10
    units = [small_workload(1510, fdot_lo=-2 * step, **kw), w]
    with P.Plan(max_sft=w.n_sft, max_bins=max(u.n_bins for u in units), max_sky=n_sky, max_fd=3, max_f=333) as p:
        call = p.compute if entry == "compute" else p.compute_noalloc
        for u, threads in zip(units, (256, 64)):
            wu, _ = to_device(u)
            out = alloc_output(u)
            call(wu, out)
            torch.cuda.synchronize()
            assert p.last_tile()["threads"] == threads, p.last_tile()
            assert twoF_error(out.twoF.cpu().numpy().ravel(), oracle_lib.fstat(u)["twoF"]).max() <= 1e-4
