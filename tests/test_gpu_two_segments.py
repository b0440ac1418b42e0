"""Gradients over several checkpoint segments, two of which are kept and the others recomputed
beside the adjoint: the same bits as from one segment, in a workspace with room for one segment
only, on another stream and from a captured graph."""

import ctypes
import re

import pytest
import torch

pytestmark = pytest.mark.gpu


# two segments (both kept), three, and many; ragged last ones; one step per segment
@pytest.mark.parametrize("N,B,H,K", [(8, 2, 9, 2), (8, 2, 17, 5), (16, 2, 10, 3), (32, 3, 13, 7), (64, 2, 21, 5), (64, 1, 5, 1), (128, 3, 11, 2),
                                     (128, 1, 12, 6), (256, 2, 9, 4), (512, 1, 7, 3), (1024, 1, 5, 2)])
def test_same_bits_however_the_segments_run(N, B, H, K):
    from paper_2602_14016_amd import Observations, Solver
    from paper_2602_14016_amd import native as nv
    print("CASE two-segments", N, B, H, K, flush=True)
    s = Solver(N, B, nu=1e-3, dt=1e-3)
    w0 = s.init_field(list(range(B)), kind=0, k0=2.5, target=0.5)
    M, steps = N // 4, sorted({0, K, H // 2, H})
    g = torch.Generator(device="cuda").manual_seed(N + H)
    vals = 0.1 * torch.randn(B, len(steps), 2, M, M, dtype=torch.float64, device="cuda", generator=g)
    obs = Observations(4, steps, vals)
    J1, g1 = s.adjoint_gradient(w0, H, obs, ckpt_every=H)
    J1, g1 = J1.clone(), g1.clone()

    def same(J, grad):
        torch.cuda.synchronize()
        assert bool((J == J1).all()) and bool((grad == g1).all())

    for _ in range(2):
        same(*s.adjoint_gradient(w0, H, obs, ckpt_every=K))
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        J, grad = s.adjoint_gradient(w0, H, obs, ckpt_every=K)
    same(J, grad)
    # a binomial schedule with few snapshots
    for slots in (1, 2, 3):
        s.set_checkpoint_slots(slots)
        same(*s.adjoint_gradient(w0, H, obs, ckpt_every=K))
    s.set_checkpoint_slots(0)
    # from stored checkpoints (nothing kept)
    ck = torch.empty(s.checkpoint_bytes(H, K), dtype=torch.uint8, device="cuda")
    s.forward(w0, H, obs, ckpt_every=K, ckpt=ck)
    assert bool((s.adjoint_from_checkpoints(ck, H, obs, K) == g1).all())
    # captured (one chain), replayed between eager calls
    J, grad = torch.empty_like(J1), torch.empty_like(g1)
    if s.workspace_bytes(H, K, len(steps), 0) < (64 << 20):
        s.adjoint_gradient_noalloc(w0, H, obs, ckpt_every=K, J=J, grad=grad)
        same(J, grad)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        J, grad = s.adjoint_gradient(w0, H, obs, ckpt_every=K)
    for _ in range(3):
        J.zero_()
        grad.zero_()
        graph.replay()
        same(J, grad)
        same(*s.adjoint_gradient(w0, H, obs, ckpt_every=K))
    # the least workspace that is accepted, one byte less refused
    lib, co = s.lib, nv.Obs(4, len(steps), (ctypes.c_int32 * len(steps))(*steps), vals.data_ptr())
    J, grad = torch.empty_like(J1), torch.empty_like(g1)
    ws = torch.empty(s.workspace_bytes(H, K, len(steps), 0) + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    call = lambda n: lib.pa_adjoint_gradient(s.ctx, ctypes.c_void_p(w0.data_ptr()), H, ctypes.byref(co),
                                             ctypes.c_void_p(J.data_ptr()), ctypes.c_void_p(grad.data_ptr()), K,
                                             ctypes.c_void_p(base), ctypes.c_size_t(n))
    assert call(256) == -2
    least = int(re.search(r"need (\d+) bytes", lib.pa_last_error().decode()).group(1))
    assert least < s.workspace_bytes(H, K, len(steps), 0) and call(least - 1) == -2
    assert call(least) == 0
    same(J, grad)
