"""The toplist selection in buffers of 2^20 and 2^21 candidates, around the
count (2^18) above which a segment is sorted as a whole: both sides of the
line, toplists on both sides of theirs, a batch with units on either side, and
repeats on one plan, each equal to the selection of the full 2F output."""
import numpy as np
import pytest

import oracle
from synth.device import to_device, alloc_output
from tests._helpers import small_workload

pytestmark = pytest.mark.gpu

HELD = 1 << 18


def _check(P, w, tf_all, o, threshold, top_k):
    tf, s, i, j, n_above = P.toplist(o)
    idx, n_ref = oracle.toplist(tf_all.astype(np.float64), threshold, top_k)
    assert n_above == n_ref
    assert np.array_equal((s.astype(np.int64) * w.n_fd + i) * w.n_f + j, idx), (threshold, top_k)
    assert np.array_equal(tf, tf_all[idx])
    assert (o.top.cpu().numpy().reshape(-1, 4)[len(idx):, 1:] == -1).all()


@pytest.mark.parametrize("cap,top_ks", [(1 << 20, (20, 4096, 4097, 65536)), (1 << 21, (20, 65536, 65537))])
def test_selection_around_the_line(cap, top_ks):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(975, n_det=1, slots=6, keep=1.0, n_sky=40, n_fd=8, n_f=1000, injections=())
    wu, _ = to_device(w)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=40, max_fd=8, max_f=1000, max_dterms=8,
                max_cands=cap) as p:
        full = alloc_output(w)
        p.compute(wu, full)
        torch.cuda.synchronize()
        tf_all = full.twoF.cpu().numpy().ravel()
        desc = np.sort(tf_all)[::-1]
        for n in (0, 3, HELD, HELD + 1, 5000, tf_all.size):
            threshold = float(desc[n - 1]) if n else float(desc[0]) * 2.0
            for top_k in top_ks:
                o = alloc_output(w, top_k=top_k, threshold=threshold, full=False)
                p.compute(wu, o)
                torch.cuda.synchronize()
                _check(P, w, tf_all, o, threshold, top_k)


def test_batch_with_units_on_either_side():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    w = small_workload(976, n_det=1, slots=6, keep=1.0, n_sky=40, n_fd=8, n_f=1000, injections=())
    wu, _ = to_device(w)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=40, max_fd=8, max_f=1000, max_dterms=8,
                max_cands=1 << 21) as p:
        full = alloc_output(w)
        p.compute(wu, full)
        torch.cuda.synchronize()
        tf_all = full.twoF.cpu().numpy().ravel()
        desc = np.sort(tf_all)[::-1]
        units = [(float(desc[n - 1]), k) for n, k in ((tf_all.size, 100), (40, 100), (HELD + 5, 30000), (9000, 500))]
        outs = [alloc_output(w, top_k=k, threshold=t, full=False) for t, k in units] + [alloc_output(w)]
        for _ in range(3):
            for o in outs[:-1]:
                o.top.fill_(-5)
            p.batch_compute([wu] * len(outs), outs)
            torch.cuda.synchronize()
            for (t, k), o in zip(units, outs):
                _check(P, w, tf_all, o, t, k)
        assert torch.equal(outs[-1].twoF, full.twoF)
