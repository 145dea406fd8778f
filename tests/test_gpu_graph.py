"""The library only enqueues kernels (and, for the overlapped schedule, event records/waits between its two
streams), so a call can be captured into a HIP graph when the caller supplies the workspace.  Replays are
checked against the eager result, several times, with eager work and synchronisations in between."""
import numpy as np
import pytest
import torch

import workloads as W
import paper_2507_01154_amd as F
from gpu_util import DEV, to_device

pytestmark = pytest.mark.gpu


def _layers(w, dims_idx):
    layers = []
    for l in dims_idx:
        spec = w.layers[l]
        X, dY = W.make_layer(w, l)
        layers.append(dict(X=to_device(X), dY=to_device(dY), d_in=spec.d_in, d_out=spec.d_out, C=w.C, sigma=w.sigma,
                           seed=w.layer_seed(l), layer=l,
                           out_grad=torch.zeros((spec.d_out, spec.d_in), device=DEV),
                           out_norms=torch.zeros((w.B,), device=DEV)))
    return layers


@pytest.mark.parametrize("schedule,case", [("scratch", "gpt2"), ("twopass", "gpt2"), ("overlap", "block2"), ("fused", "gpt2")])
def test_graph_capture_and_replay(schedule, case):
    if case == "gpt2":
        w = W.WORKLOADS["gpt2_small_mlp_up"]
        layers = _layers(w, [0])
    else:
        base = W.WORKLOADS["llama13b_block"]
        # large enough for the 256x256 path (many 256 x 256 work items per layer), which the overlapped schedule needs
        w = W.scaled_down(base, B=8, T=128, dims=[(2048, 4096), (4096, 2048), (2048, 4096)])
        layers = _layers(w, [0, 1, 2])
    arr = F.make_layers(layers)
    ws = torch.empty(F.flashdp_workspace_bytes(arr, w.B, w.T, F.BF16, schedule), dtype=torch.uint8, device=DEV)
    # eager reference (also sets the kernels' launch attributes outside the capture)
    F.flashdp_block_dp_grad(arr, w.B, w.T, F.BF16, schedule, ws)
    torch.cuda.synchronize()
    used = F.flashdp_last_schedule()
    assert used == schedule
    want = [(L["out_grad"].clone(), L["out_norms"].clone()) for L in layers]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        F.flashdp_block_dp_grad(arr, w.B, w.T, F.BF16, schedule, ws)
    assert F.flashdp_last_schedule() == used
    for rep in range(4):
        for L in layers:
            L["out_grad"].fill_(float("nan"))
            L["out_norms"].fill_(float("nan"))
        ws.random_(0, 255)                      # eager work between replays: the graph must not depend on old scratch
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for L, (og, on) in zip(layers, want):
            assert torch.equal(L["out_grad"], og), (schedule, rep)
            assert torch.equal(L["out_norms"], on), (schedule, rep)


FRESH_PROCESS = """
import torch, paper_2507_01154_amd as F
dev = "cuda:0"
out = torch.empty((4944 * 1032,), device=dev)
def layer(B, T, P, D, dt):
    torch.manual_seed(B)
    return [dict(X=torch.randn((B, T, P), device=dev).to(dt), dY=torch.randn((B, T, D), device=dev).to(dt), d_in=P, d_out=D, C=1.0,
                 sigma=0.0, seed=1, layer=0, out_grad=out)]
earlier = layer(1, 32, 1006, 4944, torch.float32)
# parks on small tiles; sums parts of the batch: each takes more than the earlier call has left, and can do with less
calls = [((5, 333), layer(5, 333, 1032, 1928, torch.bfloat16), 2048, "gemm_mfma_dma16_kernel"), ((64, 40), layer(64, 40, 1032, 1032, torch.bfloat16), 0, "gemm_tile128_kernel")]
want = []
for (B, T), L, less, kernel in calls:   # with workspaces of the caller's: the results, and the launch attributes
    size = F.flashdp_workspace_bytes(L, B, T, F.BF16, "scratch")
    for w in (2 * size, size - less):
        F.flashdp_block_dp_grad(L, B, T, F.BF16, "auto", torch.empty((w,), dtype=torch.uint8, device=dev))
        torch.cuda.synchronize()
    assert F.flashdp_last_kernel() == kernel
    want.append(out.clone())
F.flashdp_block_dp_grad(earlier, 1, 32, F.F32, "scratch")
torch.cuda.synchronize()
for ((B, T), L, less, kernel), ref in zip(calls, want):
    n = L[0]["d_in"] * L[0]["d_out"]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        F.flashdp_block_dp_grad(L, B, T, F.BF16, "auto", None)
    assert F.flashdp_last_kernel() == kernel, F.flashdp_last_kernel()
    for rep in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert float((out[:n] - ref[:n]).norm() / ref[:n].norm()) < 1e-4, rep
"""


def test_capture_on_a_library_workspace_that_holds_no_more_than_the_large_tiles_need():
    # in a process of its own: what an earlier call has left is enough for the schedule, not for what it is fastest in, and
    # must not be grown inside the capture
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", FRESH_PROCESS], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
