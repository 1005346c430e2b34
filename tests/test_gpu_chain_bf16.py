"""The walk over 64-token steps behind the bf16 forwards: edges of steps and tiles, padded sizes, routing options, the three
ways a step's decays are split over its tokens (one reference, one per half, direct), and that none of them is seen by the
tokens in front."""
import numpy as np
import pytest
import torch

from oracle import swimba_oracle as orc
from paper_2603_06938_amd import binding as sw
from paper_2603_06938_amd import synth
from gpu_util import TOL, abs_inputs, comp_tol, componentwise_excess, host, rel_errors, to_device

pytestmark = pytest.mark.gpu

CASES = [
    # B, L, H, P, N, G, E, k, h0, D, factor on dt
    (1, 1, 1, 64, 128, 1, 2, 1, False, True, 1.0),
    (2, 31, 2, 32, 32, 1, 4, 2, True, True, 1.0),
    (2, 63, 4, 64, 128, 2, 8, 2, True, False, 1.0),
    (1, 64, 2, 64, 64, 1, 8, 2, False, True, 1.0),
    (3, 65, 3, 40, 72, 1, 5, 3, True, True, 1.0),
    (2, 96, 2, 8, 8, 2, 4, 2, True, True, 1.0),
    (1, 129, 8, 64, 16, 8, 16, 2, False, True, 1.0),
    (2, 200, 4, 56, 40, 1, 64, 4, True, True, 1.0),
    (1, 577, 2, 64, 128, 1, 8, 2, True, True, 1.0),
    (2, 448, 160, 64, 128, 4, 4, 2, True, True, 1.0),     # 320 chains: a workgroup per channel tile, several groups each
    (1, 300, 160, 48, 104, 1, 4, 1, True, True, 1.0),     # 160 chains: both channel tiles in one workgroup
    (2, 333, 4, 64, 128, 2, 5, 2, True, True, 4.0),       # a reference per half for the fast heads
    (2, 333, 4, 64, 128, 2, 5, 2, True, True, 40.0),      # mostly direct
    (1, 190, 160, 64, 128, 2, 5, 2, True, True, 10.0),    # all three
    (2, 333, 4, 64, 48, 2, 5, 2, True, True, 1e-3),
    (2, 200, 160, 32, 72, 2, 4, 2, True, True, 4.0),      # 320 chains of one channel tile: two workgroups to a unit
    (3, 130, 96, 16, 128, 1, 4, 2, True, False, 40.0),    # the same, mostly direct
    (4, 67, 128, 24, 32, 4, 4, 1, False, True, 1.0),
    (2, 130, 64, 64, 128, 1, 4, 2, True, True, 10.0),     # 128 chains: a workgroup per channel tile on every unit
    (1, 130, 129, 64, 128, 1, 4, 2, True, True, 10.0),    # one more: both tiles in one
    (130, 40, 8, 8, 40, 8, 4, 2, False, True, 1.0),       # rows of less than a line in 8 groups, several groups a workgroup
    (3, 70, 7, 8, 56, 7, 4, 3, False, True, 1.0),         # in fewer groups
    (2, 70, 16, 8, 24, 16, 4, 3, False, True, 1.0),
]


def inputs(case, seed):
    B, L, H, P, N, G, E, k, with_h0, with_D, dt_scale = case
    w = synth.Workload("chain", B, L, H, P, N, G, E, k, 64, "bf16", 9)
    p = synth.make_inputs(w, seed=seed)
    # scaled step sizes, rounded to bf16 here so that both sides see the same values
    p["dt"] = torch.from_numpy(p["dt"] * np.float32(dt_scale)).to(torch.bfloat16).to(torch.float32).numpy()
    rng = np.random.default_rng(seed)
    p["D"] = rng.standard_normal(H).astype(np.float32)
    h0 = (0.1 * rng.standard_normal((B, H, P, N))).astype(np.float32) if with_h0 else None
    return p, h0


def forward(p, k, h0, with_D, chunk=64):
    d = to_device(p, "bf16")
    return sw.swimba_mixer_fwd(d["x"], d["dt"], d["A"], d["D"] if with_D else None, d["B_experts"], d["C_experts"],
                               d["router_logits"], k, chunk, None if h0 is None else torch.from_numpy(h0).to("cuda:0"),
                               want_topk=True)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d_h0%d_D%d_dt%g" % c)
def test_chain_matches_oracle(case):
    B, L, H, P, N, G, E, k, with_h0, with_D, dt_scale = case
    p, h0 = inputs(case, 100 + CASES.index(case))
    D = p["D"] if with_D else None
    out = forward(p, k, h0, with_D)
    torch.cuda.synchronize()
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], D, p["B_experts"], p["C_experts"], p["router_logits"], k, h0=h0)
    np.testing.assert_array_equal(out.topk_idx.cpu().numpy(), ref["topk_idx"])
    np.testing.assert_allclose(host(out.topk_w), ref["topk_w"], rtol=1e-5, atol=1e-30)
    q = abs_inputs(p)
    aref = orc.mixer_fwd(q["x"], q["dt"], q["A"], None if D is None else np.abs(D), q["B_experts"], q["C_experts"],
                         q["router_logits"], k, h0=None if h0 is None else np.abs(h0))
    # every term passes at most five roundings to bf16: B, x times its factor, the state, C (or C B^T), the stored y
    ey = componentwise_excess(host(out.y), ref["y"], aref["y"])
    eh = componentwise_excess(host(out.h_final), ref["h_final"], aref["h_final"])
    assert ey <= comp_tol("bf16") and eh <= comp_tol("bf16"), (ey, eh)
    if L >= 16:
        l2, linf = rel_errors(host(out.y), ref["y"], (0, 2))
        assert l2 <= TOL["bf16"] and linf <= TOL["bf16"], (l2, linf)
    # the chunk length of the call is not the chain's: the same bits
    other = forward(p, k, h0, with_D, 256)
    assert torch.equal(other.y, out.y) and torch.equal(other.h_final, out.h_final)


SEGMENTED = [
    # sequences cut into segments: few chains, long sequences (B, L, H, P, N, G, E, k, h0, D, factor on dt, chunk)
    (1, 10300, 2, 40, 72, 1, 5, 3, True, True, 1.0, 256),       # 161 steps, as many segments as the scratch holds
    (1, 10240, 3, 32, 16, 1, 4, 1, False, True, 0.05, 64),      # slow decays: every piece reaches the end
    (1, 2400, 64, 64, 128, 2, 8, 2, True, False, 1.0, 256),     # 38 steps in 3
    (1, 3072, 64, 64, 128, 1, 4, 2, True, True, 4.0, 64),       # whole chunks: pieces that no sum sees are not walked
    (1, 3072, 64, 64, 64, 8, 4, 2, True, True, 0.3, 64),
    (2, 8200, 48, 64, 128, 1, 4, 2, True, True, 1.0, 256),      # 96 chains: two rounds of segments
    (4, 6200, 36, 8, 40, 4, 4, 2, False, True, 10.0, 128),      # 144 chains; direct steps
]


@pytest.mark.parametrize("case", SEGMENTED, ids=lambda c: "B%dL%dH%dP%dN%dG%dE%dk%d_h0%d_D%d_dt%g_Q%d" % c)
def test_segments_match_oracle(case):
    B, L, H, P, N, G, E, k, with_h0, with_D, dt_scale, chunk = case
    p, h0 = inputs(case[:-1], 300 + SEGMENTED.index(case))
    D = p["D"] if with_D else None
    out = forward(p, k, h0, with_D, chunk)
    torch.cuda.synchronize()
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], D, p["B_experts"], p["C_experts"], p["router_logits"], k, h0=h0)
    q = abs_inputs(p)
    aref = orc.mixer_fwd(q["x"], q["dt"], q["A"], None if D is None else np.abs(D), q["B_experts"], q["C_experts"],
                         q["router_logits"], k, h0=None if h0 is None else np.abs(h0))
    # the roundings of the whole walk; the states that pieces leave behind are fp32
    ey = componentwise_excess(host(out.y), ref["y"], aref["y"])
    eh = componentwise_excess(host(out.h_final), ref["h_final"], aref["h_final"])
    assert ey <= comp_tol("bf16") and eh <= comp_tol("bf16"), (ey, eh)
    l2, linf = rel_errors(host(out.y), ref["y"], (0, 2))
    assert l2 <= TOL["bf16"] and linf <= TOL["bf16"], (l2, linf)


@pytest.mark.parametrize("case", [(1, 10240, 2, 40, 72, 1, 4, 2, True, True, 0.01), (1, 10496, 3, 64, 128, 1, 4, 2, True, True, 0.01)],
                         ids=["H2P40N72", "H3"])
def test_the_chunk_length_changes_no_bit_of_segments(case):
    """Scratch limits the segments of these; it is larger for smaller chunks."""
    p, h0 = inputs(case, 17)
    want = forward(p, 2, h0, True, 256)
    for chunk in (64, 128):
        got = forward(p, 2, h0, True, chunk)
        assert torch.equal(got.y, want.y) and torch.equal(got.h_final, want.h_final)


@pytest.mark.parametrize("case,chunk,segments", [((2, 200, 4, 56, 40, 1, 64, 4, True, True, 1.0), 64, 1), ((1, 3072, 64, 64, 128, 1, 4, 2, True, True, 1.0), 256, 4)],
                         ids=["whole", "segments"])
def test_stage_calls_give_the_forwards_bits(case, chunk, segments):
    """chain_mix and chain_walk are the launches of swimba_mixer_fwd where swimba_forward_path says so."""
    p, h0 = inputs(case, 18)
    k = case[7]
    d = to_device(p, "bf16")
    h = torch.from_numpy(h0).to("cuda:0")
    want = forward(p, k, h0, True, chunk)
    dims = sw.dims_of(d["x"], d["B_experts"], k, chunk)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert sw.swimba_forward_path(dims) == sw.PATH_CHAIN_BF16 and sw.swimba_forward_segments(dims) == segments
    ws = sw.alloc_workspace(dims, "cuda:0")
    y, hf = torch.empty_like(d["x"]), torch.empty_like(h)
    sw.swimba_stage_chain_mix(dims, d["dt"], d["A"], d["B_experts"], d["C_experts"], d["router_logits"], ws)
    sw.swimba_stage_chain_walk(dims, d["x"], d["D"], h, y, hf, ws)
    assert torch.equal(y, want.y) and torch.equal(hf, want.h_final)


def test_segments_final_state_over_the_initial_one():
    """In place the segments read a copy of h0: the bits of the same call out of place, every time."""
    p, h0 = inputs((1, 3100, 64, 64, 128, 1, 4, 2, True, True, 0.2), 11)
    want = forward(p, 2, h0, True, 256)
    d = to_device(p, "bf16")
    for _ in range(3):
        h = torch.from_numpy(h0).to("cuda:0")
        got = sw.swimba_mixer_fwd(d["x"], d["dt"], d["A"], d["D"], d["B_experts"], d["C_experts"], d["router_logits"], 2, 256, h,
                                  h_final=h)
        assert torch.equal(got.y, want.y) and torch.equal(h, want.h_final)


def test_segments_values_that_are_not_finite():
    """An x that is not finite reaches the tokens behind it through every later segment, and none in front."""
    p, h0 = inputs((1, 10300, 4, 64, 128, 1, 4, 2, True, True, 1.0), 12)
    base = forward(p, 2, h0, True, 256).y
    q = dict(p, x=p["x"].copy())
    q["x"][0, 3000, 1] = float("inf")
    got = forward(q, 2, h0, True, 256)
    assert torch.equal(got.y[:, :2944], base[:, :2944])
    assert torch.equal(got.y[:, :, [0, 2, 3]], base[:, :, [0, 2, 3]])
    assert not torch.isfinite(got.y[:, 3000:, 1]).any(dim=-1).any() and not torch.isfinite(got.h_final[:, 1]).any()


def test_decays_that_turn_and_growing_states():
    """dt of both signs (cs falls and rises inside a step) and of the negative one alone (the state grows)"""
    p, h0 = inputs((2, 200, 4, 64, 128, 1, 4, 2, True, True, 1.0), 7)
    rng = np.random.default_rng(8)
    turned = np.where(rng.random(p["dt"].shape) < 0.3, -0.25, 1.0).astype(np.float32)
    for f in (turned, np.float32(-0.03)):
        r = dict(p, dt=torch.from_numpy(p["dt"] * f).to(torch.bfloat16).to(torch.float32).numpy())
        out = forward(r, 2, h0, True)
        ref = orc.mixer_fwd(r["x"], r["dt"], r["A"], r["D"], r["B_experts"], r["C_experts"], r["router_logits"], 2, h0=h0)
        l2, linf = rel_errors(host(out.y), ref["y"], (0, 2))
        hl2, hlinf = rel_errors(host(out.h_final), ref["h_final"], (0, 1))
        assert max(l2, linf, hl2, hlinf) <= TOL["bf16"], (l2, linf, hl2, hlinf)


@pytest.mark.parametrize("s", [5, 31, 32, 40, 50, 64, 100])
def test_a_reference_changes_no_bit_in_front(s):
    """Larger step sizes from token s on take a step from one reference to two: tokens in front keep their bits."""
    p, h0 = inputs((1, 128, 24, 64, 128, 1, 4, 2, True, True, 1.0), 3)
    p["A"][::2] = -16.0
    bf = lambda v: torch.from_numpy(v.astype(np.float32)).to(torch.bfloat16).to(torch.float32).numpy()
    t = np.arange(128) % 64
    rng = np.random.default_rng(4)
    p["dt"] = bf(np.where(t < 32, 0.08, 0.04)[None, :, None] * (1 + 0.05 * rng.random((1, 128, 24))))
    dt = p["dt"].copy()
    dt[:, s:] = bf(0.145 * (1 + 0.05 * rng.random((1, 128 - s, 24))))
    step = 0 if s < 64 else 64
    span = lambda d, lo, hi: d[0, step + lo:step + hi, ::2].sum(0) * 16 * 1.4427
    assert span(p["dt"], 0, 64).max() < 118 and span(dt, 0, 64).min() > 122
    assert span(dt, 0, 32).max() < 118 and span(dt, 32, 64).max() < 118
    base = forward(p, 2, h0, True).y
    got = forward(dict(p, dt=dt), 2, h0, True).y
    assert torch.equal(got[:, :s], base[:, :s]) and not torch.equal(got[:, s:], base[:, s:])


@pytest.mark.parametrize("s", [1, 20, 31, 32, 33, 50, 63, 64, 100])
@pytest.mark.parametrize("shape", [(24, 64, 128), (3, 40, 72), (160, 64, 16), (300, 32, 72)],
                         ids=["H24", "H3P40N72", "H160N16", "H300P32N72"])
def test_a_direct_step_changes_no_bit_in_front(s, shape):
    """Step sizes from token s on that take its step from one reference, or one per half, to direct, to a rising cs, or to a
    value that is not finite: tokens in front keep their bits, and so do all others where the mode alone changes."""
    H, P, N = shape
    p, h0 = inputs((1, 150, H, P, N, 1, 4, 2, True, True, 1.0), 13)
    p["A"][::2] = -16.0                                   # of these heads some steps have a reference per half
    base = forward(p, 2, h0, True).y
    for value in (8.0, -0.01, float("inf"), float("nan")):
        dt = p["dt"].copy()
        dt[:, s:s + 1] = value                            # one token: its step is direct, those behind it are not
        got = forward(dict(p, dt=dt), 2, h0, True).y
        assert torch.equal(got[:, :s], base[:, :s]), value
        if not np.isfinite(value):
            assert torch.isnan(got[:, s:]).all()


def test_direct_steps_round_as_the_others_do():
    """A token that no one sees (x = 0, decay 1, first of its step's tail) but whose rising cs makes the step direct: the
    same bits everywhere."""
    p, h0 = inputs((2, 192, 24, 64, 128, 1, 4, 2, True, True, 1.0), 14)
    p["A"][:] = -np.abs(p["A"])
    q = dict(p, dt=p["dt"].copy(), x=p["x"].copy())
    p["dt"][:, 127] = 0.0
    q["dt"][:, 127] = -2.0 ** -60                         # cs and 2^(part of cs) stay what they are, but it rises
    p["x"][:, 127] = q["x"][:, 127] = 0.0
    base, got = forward(p, 2, h0, True), forward(q, 2, h0, True)
    assert torch.equal(got.y, base.y) and torch.equal(got.h_final, base.h_final)


# powers of two on (x and h0, B, C) and tokens: the scaled problem is the scaled base problem, but for the inputs' own least
# values where they come near the end of the range
MAGNITUDES = [(100, 0, 0, 330), (115, 0, 0, 330), (0, 70, -70, 200), (60, 40, -90, 200), (90, 0, 0, 10300),
              (-100, 0, 0, 330), (0, -90, 60, 200), (-50, -40, 80, 200), (-90, 0, 0, 10300)]


@pytest.mark.parametrize("sx,sb,sc,L", MAGNITUDES)
def test_magnitudes(sx, sb, sc, L):
    """Inputs far from 1 whose results are in range, at decays from slow to one that no step can hold: what the same inputs
    near 1 give."""
    H = 8
    p, h0 = inputs((1, L, H, 64, 128, 1, 4, 2, True, False, 1.0), 15)
    p["A"][:] = -16.0
    dts = np.array([1e-3, 0.01, 0.03, 0.045, 0.09, 0.16, 0.5, 3.0], np.float32)
    p["dt"] = torch.from_numpy(np.broadcast_to(dts, (1, L, H)).copy()).to(torch.bfloat16).to(torch.float32).numpy()
    base = forward(p, 2, h0, False)
    f = lambda e: np.float32(2.0 ** e)
    q = dict(p, x=p["x"] * f(sx), B_experts=p["B_experts"] * f(sb), C_experts=p["C_experts"] * f(sc))
    got = forward(q, 2, h0 * f(sx) * f(sb), False)
    y = host(got.y) / 2.0 ** (sx + sb + sc)
    h = host(got.h_final) / 2.0 ** (sx + sb)
    if min(sx, sb) >= 0 and L < 2048:
        assert np.array_equal(y, host(base.y)) and np.array_equal(h, host(base.h_final))
    # values of x and B under 2^-126 are 2^-26 of the others at most
    assert rel_errors(y, host(base.y), (0, 2))[0] < 1e-5 and rel_errors(h, host(base.h_final), (0, 1))[0] < 1e-5


@pytest.mark.parametrize("scale", [1e30, 5e37, 1e-30, 0.0])
@pytest.mark.parametrize("s", [0, 5, 40, 63, 64, 130])
def test_one_tokens_magnitude_changes_no_bit_in_front(scale, s):
    """A token whose x no factor fits takes its step to direct: the tokens in front keep their bits, those behind it are right."""
    one_token(scale, s, 24, 64, 128)


@pytest.mark.parametrize("shape", [(160, 64, 128), (300, 32, 72)], ids=["both tiles", "two workgroups a unit"])
@pytest.mark.parametrize("scale,s", [(1e30, 5), (1e30, 40), (5e37, 130), (0.0, 64)])
def test_one_tokens_magnitude_however_the_waves_share_the_walk(scale, s, shape):
    one_token(scale, s, *shape)


def one_token(scale, s, H, P, N):
    p, h0 = inputs((1, 150, H, P, N, 1, 4, 2, True, True, 1.0), 16)
    p["A"][::2] = -16.0
    p["dt"] = np.abs(p["dt"]) + np.float32(0.03125)       # most steps span 2^60 and more
    p["dt"] = torch.from_numpy(p["dt"]).to(torch.bfloat16).to(torch.float32).numpy()
    base = forward(p, 2, h0, True)
    q = dict(p, x=p["x"].copy())
    q["x"][:, s] = torch.from_numpy(np.clip(q["x"][:, s], -1, 1) * np.float32(scale)).to(torch.bfloat16).to(torch.float32).numpy()
    got = forward(q, 2, h0, True)
    assert torch.equal(got.y[:, :s], base.y[:, :s]) and torch.isfinite(got.y).all()
    ref = orc.mixer_fwd(q["x"], q["dt"], q["A"], q["D"], q["B_experts"], q["C_experts"], q["router_logits"], 2, h0=h0)
    a = abs_inputs(q)
    aref = orc.mixer_fwd(a["x"], a["dt"], a["A"], a["D"], a["B_experts"], a["C_experts"], a["router_logits"], 2, h0=np.abs(h0))
    assert componentwise_excess(host(got.y), ref["y"], aref["y"]) <= comp_tol("bf16")


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_values_that_are_not_finite_reach_no_earlier_tile(value):
    """A dt or x that is not finite leaves the tokens of the 32-token tiles in front of its own alone."""
    p, h0 = inputs((1, 192, 4, 64, 128, 1, 4, 2, True, True, 1.0), 5)
    base = forward(p, 2, h0, True).y
    for name in ("dt", "x"):
        q = dict(p)
        q[name] = p[name].copy()
        q[name][0, 100, 1] = value
        got = forward(q, 2, h0, True)
        assert torch.isfinite(got.y[:, :64]).all() and torch.equal(got.y[:, :64], base[:, :64])
        assert torch.isfinite(got.y[:, :96, 1]).all()
        assert torch.equal(got.y[:, :, [0, 2, 3]], base[:, :, [0, 2, 3]])
        assert not torch.isfinite(got.y[:, 100:, 1]).all()


def test_x_read_past_the_cache_changes_no_bit():
    """Calls whose x and y fill the last-level cache read x past it.  Two sequences do here, either of them alone does not; a
    last step of one token, heads narrower than two channel tiles."""
    B, L, H, P, N, E = 2, 3777, 160, 56, 72, 4
    assert B * L * H * P * 4 >= 256 << 20 > L * H * P * 4
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda:0").bfloat16()
    x, Be, Ce, logits = rnd(B, L, H, P), rnd(B, L, E, 1, N), rnd(B, L, E, 1, N), rnd(B, L, E)
    dt = torch.rand((B, L, H), generator=gen, device="cuda:0").mul_(0.1).bfloat16()
    A, D = -torch.linspace(0.5, 16.0, H, device="cuda:0"), torch.linspace(-1.0, 1.0, H, device="cuda:0")
    both = sw.swimba_mixer_fwd(x, dt, A, D, Be, Ce, logits, 2, 256)
    assert bool(torch.isfinite(both.y).all())
    for b in range(B):
        one = sw.swimba_mixer_fwd(x[b:b + 1], dt[b:b + 1], A, D, Be[b:b + 1], Ce[b:b + 1], logits[b:b + 1], 2, 256)
        assert torch.equal(one.y, both.y[b:b + 1]) and torch.equal(one.h_final, both.h_final[b:b + 1])
