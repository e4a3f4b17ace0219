"""The toplist selection around its chunk of 4096 candidates: counts at and
next to the chunk's edges and over several chunks, toplists shorter and longer
than the count, and more than 65536 entries (another sort), each equal to the
selection of the same call's full 2F output."""
import numpy as np
import pytest

import oracle
from synth.device import to_device, alloc_output
from tests._helpers import small_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _check(torch, w, wu, p, counts, top_ks):
    import paper_0904_1826_amd as P
    full = alloc_output(w)
    p.compute(wu, full)
    torch.cuda.synchronize()
    tf_all = full.twoF.cpu().numpy().ravel()
    desc = np.sort(tf_all)[::-1]
    for n in counts:
        threshold = float(desc[n - 1]) if n else float(desc[0]) * 2.0
        for top_k in top_ks:
            o = alloc_output(w, top_k=top_k, threshold=threshold, full=False)
            p.compute(wu, o)
            torch.cuda.synchronize()
            tf, s, i, j, n_above = P.toplist(o)
            idx, n_ref = oracle.toplist(tf_all.astype(np.float64), threshold, top_k)
            assert n_above == n_ref and n_ref >= n
            assert np.array_equal((s.astype(np.int64) * w.n_fd + i) * w.n_f + j, idx), (n, top_k)
            assert np.array_equal(tf, tf_all[idx])
            rest = o.top.cpu().numpy().reshape(-1, 4)[len(idx):]
            assert (rest[:, 1:] == -1).all()


@pytest.mark.parametrize("top_k", [1, 37, 4097, 20000])
def test_selection_at_chunk_edges(torch_cuda, top_k):
    import paper_0904_1826_amd as P
    w = small_workload(970, n_sky=4, n_fd=5, n_f=700, slots=12, injections=((1, 2, 333, 14.0),))
    wu, _ = to_device(w)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=4, max_fd=5, max_f=700, max_dterms=8) as p:
        _check(torch_cuda, w, wu, p, (0, 1, 2, 255, 257, 4095, 4096, 4097, 8192, 8193, 14000), (top_k,))


def test_selection_of_more_than_65536(torch_cuda):
    import paper_0904_1826_amd as P
    w = small_workload(971, n_sky=12, n_fd=8, n_f=900, slots=6, injections=())
    wu, _ = to_device(w)
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=12, max_fd=8, max_f=900, max_dterms=8,
                max_cands=100000) as p:
        _check(torch_cuda, w, wu, p, (3, 70000), (1000, 65536, 65537, 80000))
