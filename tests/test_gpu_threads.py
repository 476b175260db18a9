"""Two host threads on streams of their own, calling kernels whose dynamic LDS depends on the descriptor
(Sinkhorn-Knopp iterations; logits of the gradient on x; permutations kept) with different needs: every
call gets what it asks for, whichever thread was the last to set the limit."""
import threading

import pytest
import torch

import synth_inputs as si
from gpu_harness import GpuLayer, desc_for

pytestmark = pytest.mark.gpu

PAIRS = [(dict(n=5, C=64, T=200, res_mode="sk", sk_iters=32), dict(n=5, C=64, T=200, res_mode="sk", sk_iters=9)),
         (dict(n=4, C=64, T=200, res_mode="sk", sk_iters=32), dict(n=4, C=64, T=200, res_mode="sk", sk_iters=11)),
         (dict(n=8, C=40, T=70, res_mode="subset", n_perm=120), dict(n=8, C=40, T=70, res_mode="subset", n_perm=64))]


@pytest.mark.parametrize("pair", PAIRS, ids=["sk_n5", "sk_n4", "subset_n8"])
def test_calls_of_two_threads(pair):
    layers, want = [], []
    for form in pair:
        wl = si.Workload("thread", **form)
        inp = si.make_inputs(wl, seed=29, device="cuda")
        L = GpuLayer(desc_for(wl, perm=inp.get("perm")), inp)
        L.step()
        torch.cuda.synchronize()
        layers.append(L)
        want.append([t.clone() for t in (L.h, L.g_x, L.g_W, L.g_b, L.g_alpha)])
    failed = []

    def work(L, stream):
        try:
            with torch.cuda.stream(stream):
                for _ in range(100):
                    L.step()
            stream.synchronize()
        except Exception as e:
            failed.append(e)

    threads = [threading.Thread(target=work, args=(L, torch.cuda.Stream())) for L in layers]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for L, w in zip(layers, want):
        for a, b in zip((L.h, L.g_x, L.g_W, L.g_b, L.g_alpha), w):
            assert torch.equal(a, b)
