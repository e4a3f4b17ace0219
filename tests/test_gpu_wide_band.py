"""A unit whose band has 2^20 bins and more, with templates in its last
columns, in one batch with ordinary units whose tiles are the majority of
every launch: each unit's 2F equals what fstat_compute gives for it alone,
and the oracle's, with tiles of one sky point and of two."""
import numpy as np
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import replace, small_workload, twoF_error

pytestmark = pytest.mark.gpu


def widened(w, below):
    """The same unit with `below` columns of zeros before its band."""
    x = np.zeros((w.n_sft, below + w.n_bins), dtype=w.sft.dtype)
    x[:, below:] = w.sft
    assert w.k_first >= below
    return replace(w, sft=x, k_first=w.k_first - below)


@pytest.mark.parametrize("n_sky", [3, 8])
def test_wide_band_in_a_batch_of_ordinary_units(oracle_lib, n_sky):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    kw = dict(n_det=1, slots=6, keep=1.0, n_sky=n_sky, n_fd=8, fdot_lo=-1e-10, f0=700.0, dterms=8,
              injections=((1, 2, 90, 15.0),))
    ws = [small_workload(1100 + k, n_f=520, **kw) for k in range(5)]
    ws.append(widened(small_workload(1110, n_f=260, **kw), 1 << 20))
    devs = [to_device(w)[0] for w in ws]
    outs, alone = ([alloc_output(w) for w in ws] for _ in range(2))
    with P.Plan(max_sft=6, max_bins=max(w.n_bins for w in ws), max_sky=n_sky, max_fd=8, max_f=520) as p:
        p.batch_compute(devs, outs)
        for d, o in zip(devs, alone):
            p.compute(d, o)
        torch.cuda.synchronize()
    for w, o, a in zip(ws, outs, alone):
        e = twoF_error(o.twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"])
        assert e.max() <= 1e-4, (w.name, e.max())
        assert torch.equal(o.twoF, a.twoF), w.name
