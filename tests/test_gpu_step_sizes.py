"""Decode steps at the edges of the one-launch kernel: every state size it takes and one it does not, head
dimensions that leave a register row or a block partly empty, 16 and 17 experts and 16 and 17 tokens (with and
without routing inside the update), tied logits; against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import swimba_oracle as orc
from paper_2603_06938_amd import binding as sw
from paper_2603_06938_amd import synth
from gpu_util import TOL, host, rel_errors, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    # B, L, H, P, N, G, E, k, io
    (2, 1, 4, 64, 16, 2, 16, 4, "bf16"),
    (1, 16, 3, 24, 32, 1, 16, 16, "f32"),
    (2, 17, 2, 65, 64, 1, 5, 2, "bf16"),
    (1, 3, 2, 100, 256, 2, 17, 3, "f32"),
    (2, 33, 4, 64, 128, 4, 40, 2, "bf16"),
    (40, 1, 64, 64, 128, 8, 8, 2, "bf16"),     # more than one round of blocks
    (2, 2, 2, 1, 128, 1, 1, 1, "f32"),
    (1, 6, 2, 64, 80, 1, 8, 2, "bf16"),        # a state size with an update launch per token
    # rows that come mixed: four, five and sixteen tokens, whole and short groups of sixteen, every number of registers
    (3, 4, 4, 40, 16, 2, 17, 2, "f32"),
    (2, 5, 2, 64, 256, 1, 17, 2, "bf16"),
    (1, 32, 4, 64, 16, 1, 8, 4, "bf16"),
    (5, 64, 16, 30, 32, 2, 8, 2, "f32"),
    (12, 31, 32, 64, 64, 1, 8, 2, "bf16"),
    (8, 18, 24, 64, 128, 1, 20, 2, "f32"),
    (64, 17, 16, 64, 128, 1, 4, 1, "bf16"),
    (40, 16, 16, 33, 256, 1, 18, 1, "f32"),
    (64, 64, 8, 2, 64, 8, 2, 1, "f32"),        # four pieces of the mixed rows per lane, two of them past the end
    (64, 64, 4, 2, 33, 4, 3, 2, "bf16"),       # the same a column at a time
], ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d%s" % c)
def test_step_sizes_match_oracle(cfg):
    B, L, H, P, N, G, E, k, io = cfg
    w = synth.Workload("sizes", B, L, H, P, N, G, E, k, 0, io, 7)
    p = synth.make_decode_inputs(w, seed=sum(cfg[:8]))
    p["router_logits"] = np.round(p["router_logits"] * 2) / 2          # ties: the lower index goes first
    p["D"] = np.linspace(-1, 1, H).astype(np.float32)
    d = to_device(p, io)
    args = [d[q] for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    if L == 1:
        args = [a[:, 0].contiguous() if i not in (2, 3) else a for i, a in enumerate(args)]
        out = sw.swimba_step(d["state"], *args, k, want_topk=True)
    else:
        out = sw.swimba_step_multi(d["state"], *args, k, want_topk=True)
    torch.cuda.synchronize()
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], p["D"], p["B_experts"], p["C_experts"], p["router_logits"], k,
                        h0=p["state"].astype(np.float64))
    np.testing.assert_array_equal(out.topk_idx.cpu().numpy().reshape(B, L, k), ref["topk_idx"])
    assert out.state.data_ptr() == d["state"].data_ptr()
    l2, linf = rel_errors(host(out.state), ref["h_final"], (0, 1))
    assert l2 <= 1e-5 and linf <= 1e-5, ("state", l2, linf)   # fp32 arithmetic on both io types
    # whole-output norm: with few tokens and channels a (batch, head) slice is a handful of cancelling scalars
    l2, linf = rel_errors(host(out.y).reshape(B, L, H, P), ref["y"], ())
    assert l2 <= TOL[io] and linf <= TOL[io], ("y", l2, linf)


@pytest.mark.parametrize("E", [8, 17])
@pytest.mark.parametrize("L", [17, 33, 64])
def test_the_state_crosses_memory_once(L, E):
    """However many tokens a call has, two kernels run: one that routes and mixes, one that updates the state."""
    x = torch.randn(2, L, 4, 64, device="cuda:0")
    dt, lg = torch.rand(2, L, 4, device="cuda:0"), torch.randn(2, L, E, device="cuda:0")
    A, Be = -torch.ones(4, device="cuda:0"), torch.randn(2, L, E, 1, 128, device="cuda:0")
    state = torch.zeros(2, 4, 64, 128, device="cuda:0")
    dims = sw.make_dims(2, L, 4, 64, 128, 1, E, 2, 0, torch.float32)
    ws = torch.empty(sw.swimba_step_multi_workspace_bytes(dims), dtype=torch.uint8, device="cuda:0")
    y = torch.empty_like(x)
    call = lambda: sw.swimba_step_multi(state, x, dt, A, None, Be, Be, lg, 2, y=y, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t()
    assert sw._load().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == 2
