"""Contexts on two GPUs of one process: every call runs on its context's own
GPU, whichever the calling thread used last."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


def test_paths_of_a_context_on_another_gpu(oracle, inputs):
    import torch
    from paper_1504_02577_amd import panther as pm

    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    g = inputs.ba_graph(1000, 5)
    A, B = pm.Panther(0), pm.Panther(1)
    for P, seed in ((A, 3), (B, 4)):
        P.load_graph(g)
        P.sample_paths(5, 3001, seed)
    for P, dev, seed in ((A, 0, 3), (B, 1, 4)):
        want = oracle.walk(g, 5, 3001, seed)
        for current in (0, 1):
            print(f"case: paths of GPU {dev} with GPU {current} current", flush=True)
            out = torch.empty((3001, 6), dtype=torch.int32, device=f"cuda:{dev}")
            torch.cuda.synchronize(dev)
            torch.cuda.set_device(current)
            P._check(pm.panther_get_paths(P.h, ctypes.c_void_p(out.data_ptr()), pm.PANTHER_MEM_DEVICE))
            assert (out.cpu().numpy() == want).all()
            torch.cuda.set_device(current)
            assert (P.paths() == want).all()
    torch.cuda.set_device(0)
    A.close()
    B.close()
