"""Small units on the GPU: one wave per (sky point, spindown, 64 frequencies)
instead of interp tiles.  The arithmetic per template and SFT is the tiles',
in the same order, so 2F, Fa and Fb must equal theirs (forced through the
tile cache) bit for bit, and the oracle's within its tolerance: around the
edges of a wave's 64 frequencies, of the groups of SFTs it loads ahead and
of the blocks of 64 SFTs whose values it keeps in LDS, for every spindown
count of a work-group's four waves, with and without pairs of sky points."""
import numpy as np
import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu

# (SFTs, sky points, spindowns, frequencies)
SHAPES = [(2, 1, 1, 1), (3, 1, 1, 63), (4, 2, 2, 64), (5, 1, 3, 65), (8, 3, 4, 129), (9, 5, 5, 64), (63, 4, 3, 70),
          (64, 1, 9, 191), (65, 7, 2, 257), (66, 9, 3, 65), (127, 1, 1, 300), (129, 6, 7, 66), (200, 1, 17, 130)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("coef,phase,storage", [("f32", "fp64", "c64"), ("f32", "split", "bf16"), ("f16", "fp64", "fp16")])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_wave_kernel_equals_tiles_and_oracle(torch_cuda, oracle_lib, tmp_path, shape, coef, phase, storage):
    import paper_0904_1826_amd as P
    torch = torch_cuda
    n_sft, n_sky, n_fd, n_f = shape
    n_det = 1 if n_sft < 4 or n_sft % 2 else 2
    w = small_workload(950 + n_sft, n_det=n_det, slots=n_sft // n_det, keep=1.0, n_sky=n_sky, n_fd=n_fd, n_f=n_f,
                       dterms=8, fdot_lo=-1e-9 if n_fd > 1 else 0.0, injections=((0, 0, n_f // 2, 12.0),))
    assert w.n_sft == n_sft
    wu, deq = to_device(w, storage)
    cache = tmp_path / "tiles.txt"
    s_, c_ = P.STORAGE[storage], 1 if coef == "f16" else 0
    cache.write_text(f"s{s_}_d8_k0_c{c_} 8 {5 if c_ else 4} 0 256\nbatch_s{s_}_c{c_} 8 256 256 256\n")
    outs = []
    for tuned in (False, True):
        o = alloc_output(w, fafb=True, top_k=5, threshold=4.0)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=n_fd, max_f=n_f, max_dterms=8,
                    storage=storage, phase=phase, coef=coef) as p:
            if tuned:
                p.autotune(wu, o, cache_path=str(cache))
            p.compute(wu, o)
            torch.cuda.synchronize()
            assert p.last_tile()["nf_reg"] == (8 if tuned else 1)
        outs.append(o)
    for name in ("twoF", "fa", "fb", "n_above"):
        assert torch.equal(getattr(outs[0], name), getattr(outs[1], name)), name
    a, b = P.toplist(outs[0]), P.toplist(outs[1])
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    e = twoF_error(outs[0].twoF.cpu().numpy().ravel(), oracle_lib.fstat(w, sft=deq)["twoF"])
    assert e.max() <= (5e-3 if coef == "f16" else 1e-4)


def test_units_beyond_the_rule_keep_their_tiles(torch_cuda):
    """Eight spindowns cross at about 5.6e5 templates; one spindown has no efficient tile at any size."""
    import paper_0904_1826_amd as P
    torch = torch_cuda
    for n_sky, n_fd, n_f, wave in ((40, 8, 1536, True), (60, 8, 1536, False), (400, 1, 2048, True)):
        w = small_workload(990, n_det=1, slots=6, keep=1.0, n_sky=n_sky, n_fd=n_fd, n_f=n_f, dterms=8,
                           fdot_lo=-1e-9 if n_fd > 1 else 0.0, injections=())
        wu, _ = to_device(w)
        o = alloc_output(w)
        with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=n_fd, max_f=n_f, max_dterms=8) as p:
            p.compute(wu, o)
            torch.cuda.synchronize()
            assert (p.last_tile()["nf_reg"] == 1) == wave, (n_sky, n_fd, n_f)
