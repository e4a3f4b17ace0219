"""D-hat-phi one ulp below an integer in every (template, SFT) pair, with a band
that holds exactly the windows of the grid: every form of the interp kernel
must take the k* that the band check and the oracle take, since the bin beyond
has no window in the band (its coefficients are zeros).  T_sft and df are
powers of two, the detector is at rest and the spindowns are 0, so
D-hat-phi = 1024 f0 + j - ulp exactly, from the lowest of its binades to the
one where its words are read."""
import numpy as np
import pytest

import synth
from synth.device import to_device, alloc_output
from tests._helpers import replace, twoF_error

pytestmark = pytest.mark.gpu

N_F = 300


def edge_workload(f0, n_fd=8):
    """f0: an integer; the grid starts one ulp of f0 below it."""
    below = float(np.nextafter(f0, 0.0))
    w = synth.make_workload(f"edge-{f0}", seed=830, n_det=1, slots_per_det=12, keep_frac=1.0, jitter=60.0,
                            t_sft=1024.0, f0=below, n_f=N_F, n_sky=3, n_fd=n_fd, fdot_lo=0.0, fdot_hi=0.0, dterms=8,
                            injections=())
    w = replace(w, vel=np.zeros_like(w.vel))
    first = int(1024 * f0) - 1                       # k* of the first template; the last one's is first + N_F - 1
    lo, hi = first - w.dterms + 1, first + N_F - 1 + w.dterms
    a = lo - w.k_first
    assert a >= 0 and hi < w.k_first + w.n_bins
    return replace(w, sft=np.ascontiguousarray(w.sft[:, a:a + hi - lo + 1]), k_first=lo)


FORMS = {"direct": dict(kernel="direct"), "wave": {}, "tile": {}, "wave16": dict(coef="f16"), "tile16": dict(coef="f16"),
         "batch": {}, "batch16": dict(coef="f16"), "noalloc": {}}


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("f0", [60, 100, 500, 1100, 1400, 2500])
def test_tight_band_one_ulp_below_an_integer(oracle_lib, tmp_path, f0, form):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = edge_workload(f0)
    wu, _ = to_device(w)
    out = alloc_output(w)
    cache = tmp_path / "tiles.txt"
    cache.write_text("s0_d8_k0_c0 8 4 0 256\ns0_d8_k0_c1 8 5 0 256\nbatch_s0_c0 8 256 256 256\n"
                     "batch_s0_c1 8 256 256 256\n")
    print(form, f0, w.k_first, w.n_bins, flush=True)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=3, max_fd=8, max_f=N_F, max_dterms=8, **FORMS[form]) as p:
        if form.startswith("tile"):
            p.autotune(wu, out, cache_path=str(cache))
        if form.startswith("batch"):
            p.batch_compute([wu], [out])
        elif form == "noalloc":
            p.compute_noalloc(wu, out)
        else:
            p.compute(wu, out)
        torch.cuda.synchronize()
        if form.startswith(("tile", "wave")):
            assert (p.last_tile()["nf_reg"] == 1) == form.startswith("wave")
    ref = oracle_lib.fstat(w)["twoF"]
    e = twoF_error(out.twoF.cpu().numpy().ravel(), ref)
    assert e.max() <= (5e-3 if form.endswith("16") else 1e-4), (int(e.argmax()) % N_F, e.max())


def test_words_and_conversions_agree(oracle_lib):
    """A unit whose words are read when it runs alone, batched with one outside
    that binade (then both are converted): the same 2F bit for bit, also one
    ulp below an integer."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    form = lambda ws: P.fstat_slot_form([(w.df, w.dfdot, w.t_sft, w.k_first, w.n_bins, 1e7, 10) for w in ws])
    ws = [edge_workload(1100), edge_workload(100)]
    assert form(ws[:1]) == 2 and form(ws) == 1
    devs = [to_device(w)[0] for w in ws]
    outs, alone = ([alloc_output(w) for w in ws] for _ in range(2))
    with P.Plan(max_sft=ws[0].n_sft, max_bins=max(w.n_bins for w in ws), max_sky=3, max_fd=8, max_f=N_F) as p:
        p.batch_compute(devs, outs)
        for d, o in zip(devs, alone):
            p.batch_compute([d], [o])
        torch.cuda.synchronize()
    for w, o, a in zip(ws, outs, alone):
        assert torch.equal(o.twoF, a.twoF)
        assert twoF_error(o.twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"]).max() <= 1e-4
