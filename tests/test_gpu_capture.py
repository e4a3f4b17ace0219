"""Calls that wait for the band check cannot run on a stream under capture:
the check they would read is not this call's.  They say so (FSTAT_E_DEVICE)
and leave the outputs, the capture and the plan as they were."""
import ctypes

import pytest

from synth.device import to_device, alloc_output
from tests._helpers import small_workload, twoF_error

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(l.split()[-1] for l in f if "libamdhip64" in l))


@pytest.mark.parametrize("entry,n_sky", [("compute", 2), ("compute", 6), ("noalloc", 2), ("batch", 2),
                                         ("semicoherent", 2)])
def test_refused_under_capture_and_whole_again_after(oracle_lib, entry, n_sky):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1826_amd as P
    hip = _hip()
    w = small_workload(1700, n_det=2, slots=20, keep=1.0, n_sky=n_sky, n_fd=3, n_f=200,
                       injections=((1, 1, 90, 12.0),))
    wu, _ = to_device(w)
    out = alloc_output(w)
    s = torch.cuda.Stream()
    with P.Plan(max_sft=w.n_sft, max_bins=w.n_bins, max_sky=n_sky, max_fd=3, max_f=200) as p:
        call = {"compute": lambda: p.compute(wu, out, stream=s),
                "noalloc": lambda: p.compute_noalloc(wu, out, stream=s),
                "batch": lambda: p.batch_compute([wu], [out], stream=s),
                "semicoherent": lambda: p.semicoherent([wu], out, stream=s)}[entry]
        call()                                       # a result of an earlier call is there to be misread
        torch.cuda.synchronize()
        out.twoF.fill_(-1.0)
        torch.cuda.synchronize()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 1) == 0      # thread-local
        try:
            with pytest.raises(P.FstatError) as e:
                call()
        finally:
            graph = ctypes.c_void_p()
            end = hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph))
            if graph.value:
                hip.hipGraphDestroy(graph)
            hip.hipGetLastError()
        assert e.value.code == P.FSTAT_E_DEVICE and end == 0
        torch.cuda.synchronize()
        assert bool((out.twoF == -1.0).all())
        for _ in range(2):
            call()
            torch.cuda.synchronize()
            assert twoF_error(out.twoF.cpu().numpy().ravel(), oracle_lib.fstat(w)["twoF"]).max() <= 1e-4
            out.twoF.fill_(-1.0)
