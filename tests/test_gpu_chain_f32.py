"""The fp32 chain at its edges: lengths around its steps of 64 tokens, one to 64 segments with a short and an
empty last one, head and state sizes around its tiles of 32, one and two state tiles per wave, 16 and 17
experts, bf16 io at sizes outside the bf16 kernels, and the final state written over the initial one;
against the oracle in double.

Tolerance: an output is a sum of at most N + 64 products per step with the state carried in fp32 over the steps it
remembers, 16 for the slowest head (A = -1, dt = 1e-3), so its relative error stays below about
sqrt(16 * (256 + 64)) * 2^-24 = 4e-6.  The factors exp(cs_i - cs_j) come from sums over a step of up to 81 (117 in powers
of two), which fp32 holds to 117 * 2^-24: another 117 * ln 2 * 2^-24 = 5e-6.  Together 1e-5 for the whole-output norm
(seen: 3e-8 in y, 7e-7 in the state); bf16 io: y's rounding, 2^-8."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import swimba_oracle as orc
from paper_2603_06938_amd import binding as sw
from paper_2603_06938_amd import synth
from gpu_util import host, to_device

pytestmark = pytest.mark.gpu
BAR = {"f32": 1e-5, "bf16": 2.0 ** -8}


def inputs(B, L, H, P, N, G, E, k, io):
    w = synth.Workload("chain", B, L, H, P, N, G, E, k, 64, io, 7)
    p = synth.make_inputs(w, seed=B + 3 * L + 5 * H + 7 * P + 11 * N + 13 * E)
    p["D"] = np.linspace(-1, 1, H).astype(np.float32)
    h0 = (0.1 * np.random.default_rng(L).standard_normal((B, H, P, N))).astype(np.float32)
    return p, h0


def rel(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def check(y, hf, p, k, h0, io):
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], p["D"], p["B_experts"], p["C_experts"], p["router_logits"], k,
                        h0=h0)
    assert rel(host(y), ref["y"]) <= BAR[io]
    assert rel(host(hf), ref["h_final"]) <= 1e-5


@pytest.mark.parametrize("cfg", [
    # B, L, H, P, N, G, E, k, io
    (1, 1, 1, 1, 1, 1, 1, 1, "f32"),
    (2, 63, 2, 31, 33, 1, 4, 2, "f32"),
    (2, 64, 4, 32, 32, 2, 16, 3, "f32"),
    (1, 65, 3, 33, 126, 3, 17, 2, "f32"),
    (1, 511, 2, 64, 128, 1, 8, 2, "f32"),
    (1, 513, 2, 40, 129, 1, 8, 2, "f32"),      # two state tiles per wave
    (1, 577, 4, 32, 256, 2, 8, 2, "f32"),      # ten steps in five segments
    (1, 1100, 2, 64, 64, 1, 5, 5, "f32"),      # 18 steps in nine segments
    (1, 2100, 2, 16, 48, 1, 8, 2, "f32"),      # 33 steps in 32: two each, the last fifteen empty, one short
    (1, 16623, 1, 16, 16, 1, 8, 2, "f32"),     # 260 steps in 64: five each, the last twelve empty
    (2, 8200, 2, 33, 20, 1, 4, 2, "f32"),      # 129 steps in 32, a slice of one channel
    (2, 2050, 48, 8, 12, 2, 4, 2, "f32"),      # 96 chains in eight segments, more steps than mix in four parts
    (1, 600, 2, 24, 80, 1, 8, 2, "f32"),
    (2, 30, 3, 40, 9, 1, 4, 2, "f32"),         # one tile row, a quarter of its blocks a wave
    (3, 9, 2, 64, 64, 1, 4, 2, "f32"),         # two waves to a tile, blocks without a token
    (1, 130, 2, 64, 65, 1, 4, 2, "f32"),       # three tiles: a wave each
    (1, 600, 2, 128, 60, 1, 8, 2, "bf16"),     # outside the bf16 kernels
    (1, 70, 2, 20, 160, 2, 8, 2, "bf16"),
], ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d%s" % c)
def test_chain_sizes(cfg):
    k, io = cfg[7], cfg[8]
    p, h0 = inputs(*cfg)
    d = to_device(p, io)
    args = [d[q] for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    for h in (None, h0):
        out = sw.swimba_mixer_fwd(*args, k, 64, None if h is None else torch.from_numpy(h).cuda())
        torch.cuda.synchronize()
        check(out.y, out.h_final, p, k, h, io)


def test_growing_state():
    """A positive A (and a negative dt) is outside the model but not refused: the factors of M exceed 1."""
    p, h0 = inputs(1, 200, 4, 32, 64, 1, 8, 2, "f32")
    p["A"] = np.array([0.5, -0.5, 2.0, -2.0], np.float32)
    p["dt"][:, 50:60] *= -1
    d = to_device(p, "f32")
    args = [d[q] for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    out = sw.swimba_mixer_fwd(*args, 2, 64, torch.from_numpy(h0).cuda())
    torch.cuda.synchronize()
    check(out.y, out.h_final, p, 2, h0, "f32")


def test_final_state_over_the_initial_one():
    B, L, H, P, N, G, E, k = 2, 700, 4, 64, 128, 1, 8, 2
    p, h0 = inputs(B, L, H, P, N, G, E, k, "f32")
    d = to_device(p, "f32")
    state = torch.from_numpy(h0).cuda()
    y = torch.empty_like(d["x"])
    dims = sw.dims_of(d["x"], d["B_experts"], k, 64)
    ws = sw.alloc_workspace(dims, "cuda:0")
    ptrs = [d[q].data_ptr() for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    status = sw._load().swimba_mixer_fwd(ctypes.byref(dims), *ptrs, state.data_ptr(), y.data_ptr(), state.data_ptr(),
                                         None, None, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert status == 0
    torch.cuda.synchronize()
    check(y, state, p, k, h0, "f32")


@pytest.mark.parametrize("cfg", [
    (1, 2100, 2, 16, 48, 1, 8, 2, "f32"),      # two steps a segment, nearly half of them empty
    (2, 700, 4, 64, 128, 1, 8, 2, "f32"),
    (1, 577, 4, 33, 240, 2, 8, 2, "f32"),      # a slice of one channel, two state tiles per wave
    (1, 1100, 1, 24, 18, 1, 8, 2, "bf16"),
    (1, 60, 1, 24, 18, 1, 8, 2, "f32"),        # one segment
], ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d%s" % c)
def test_a_state_in_place_gives_the_same_bits(cfg):
    """The sequence is walked in the same segments whether or not the final state goes over the initial one."""
    k = cfg[7]
    p, h0 = inputs(*cfg)
    d = to_device(p, cfg[8])
    args = [d[q] for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    apart = sw.swimba_mixer_fwd(*args, k, 64, torch.from_numpy(h0).cuda())
    state = torch.from_numpy(h0).cuda()
    over = sw.swimba_mixer_fwd(*args, k, 64, state, h_final=state)
    torch.cuda.synchronize()
    assert over.h_final.data_ptr() == state.data_ptr()
    assert torch.equal(over.y, apart.y) and torch.equal(state, apart.h_final)


WHICH = ["x_inf", "x_nan", "dt_inf", "dt_nan", "B_nan", "C_inf"]


@pytest.mark.parametrize("L,j", [(600, 5), (600, 31), (600, 32), (600, 63), (600, 64), (600, 80), (600, 330), (20, 5)])
@pytest.mark.parametrize("which", WHICH)
def test_values_that_are_not_finite_stay_causal(which, L, j):
    """Uninitialised padding behind a sequence, say: tokens in front of it, other channels (x), other heads (dt)
    and other sequences keep their values; its own token does not hide it."""
    stays_causal((2, L, 4, 40, 48, 1, 8, 2, "f32"), which, j)       # 600 tokens: five segments of two steps


@pytest.mark.parametrize("N", [20, 65, 200], ids=["four waves a tile", "one", "two tiles a wave"])
@pytest.mark.parametrize("L,j", [(600, 10), (600, 63), (600, 90), (20, 5)])
@pytest.mark.parametrize("which", WHICH)
def test_values_that_are_not_finite_stay_causal_however_the_waves_share_the_state(which, L, j, N):
    stays_causal((2, L, 4, 40, N, 1, 8, 2, "f32"), which, j)


def stays_causal(cfg, which, j):
    B, L, H, P = cfg[:4]
    p, h0 = inputs(*cfg)
    d = to_device(p, "f32")
    names = ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")
    h = torch.from_numpy(h0).cuda()
    clean = sw.swimba_mixer_fwd(*[d[q] for q in names], 2, 64, h)
    bad = float("inf") if which.endswith("inf") else float("nan")
    hit = torch.zeros(B, L, H, P, dtype=torch.bool, device="cuda:0")
    if which[0] == "x":
        d["x"][1, j, 2, 33] = bad
        hit[1, j:, 2, 33] = True
    elif which[0] == "d":
        d["dt"][1, j, 2] = bad
        hit[1, j:, 2] = True
    else:
        d["B_experts" if which[0] == "B" else "C_experts"][1, j] = bad
        hit[1, j:(None if which[0] == "B" else j + 1)] = True
    out = sw.swimba_mixer_fwd(*[d[q] for q in names], 2, 64, h)
    torch.cuda.synchronize()
    assert not torch.isfinite(out.y[1, j][hit[1, j]]).any()
    kept = ~hit
    assert torch.isfinite(out.y[kept]).all()
    assert rel(host(out.y[kept]), host(clean.y[kept])) <= 1e-6     # the sums are taken in another order


@pytest.mark.parametrize("cfg", [
    # B, L, H, P, N, G, E, k, io: steps that are not full, one and two tile rows, with and without other steps
    (3, 1, 4, 8, 16, 2, 17, 2, "f32"),
    (2, 7, 3, 33, 130, 3, 16, 2, "bf16"),
    (2, 8, 2, 64, 128, 1, 256, 3, "f32"),
    (70, 9, 2, 8, 8, 1, 5, 2, "f32"),          # more steps than four workgroups share
    (2, 16, 2, 20, 32, 1, 8, 2, "f32"),
    (70, 17, 4, 4, 40, 4, 40, 2, "f32"),
    (2, 31, 2, 16, 16, 1, 8, 2, "f32"),
    (70, 32, 2, 16, 60, 2, 8, 2, "bf16"),
    (2, 33, 2, 32, 32, 1, 8, 2, "f32"),
    (70, 49, 2, 8, 16, 1, 33, 2, "f32"),
    (2, 145, 2, 40, 48, 1, 8, 2, "f32"),
    (600, 5, 4, 4, 8, 4, 17, 2, "f32"),        # two groups share a workgroup
    (160, 100, 8, 2, 4, 8, 8, 2, "f32"),
    (1, 60, 2, 4, 4, 1, 256, 8, "f32"),        # logits that need more LDS than the rows
], ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d%s" % c)
def test_steps_that_are_not_full(cfg):
    """From a workspace of NaN: the chain reads nothing that was not written for it, and sums nothing that is not finite."""
    k, io = cfg[7], cfg[8]
    p, h0 = inputs(*cfg)
    d = to_device(p, io)
    args = [d[q] for q in ("x", "dt", "A", "D", "B_experts", "C_experts", "router_logits")]
    ws = sw.alloc_workspace(sw.dims_of(d["x"], d["B_experts"], k, 64), "cuda:0")
    ws.fill_(255)
    out = sw.swimba_mixer_fwd(*args, k, 64, torch.from_numpy(h0).cuda(), workspace=ws, want_topk=True)
    torch.cuda.synchronize()
    check(out.y, out.h_final, p, k, h0, io)
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], p["D"], p["B_experts"], p["C_experts"], p["router_logits"], k, h0=h0)
    np.testing.assert_array_equal(out.topk_idx.cpu().numpy(), ref["topk_idx"])
