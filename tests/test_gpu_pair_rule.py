"""The choice between tiles of one and of two sky points: a unit whose paired
work-groups leave the device half empty in their last round runs single
tiles, one that fills it runs paired ones, and a tuned tile runs paired
whatever the size.  The results do not depend on the choice."""
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sky,n_fd,n_f,paired", [(61, 5, 4001, False), (150, 8, 3600, False), (256, 8, 3071, True)])
def test_pairs_by_fill_of_the_device(n_sky, n_fd, n_f, paired, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(1010, n_det=1, slots=6, keep=1.0, n_sky=n_sky, n_fd=n_fd, n_f=n_f, f0=60.0, injections=())
    wu, _ = to_device(w)
    cache = tmp_path / "tiles.txt"
    cache.write_text("s0_d8_k0_c0 8 4 0 256\n")
    outs = []
    for tuned in (False, True):
        o = alloc_output(w)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=n_fd, max_f=n_f) as p:
            if tuned:
                p.autotune(wu, o, cache_path=str(cache))
            p.compute(wu, o)
            torch.cuda.synchronize()
            t = p.last_tile()
            assert t["nf_reg"] == 8 and (t["pair_seg"] > 0) == (paired or tuned), t
        outs.append(o)
    assert torch.equal(outs[0].twoF, outs[1].twoF)
