"""GPU parity of the routed expert in-projection (the step upstream of the mixer) against
the oracle, and of projection + mixer end to end."""
import numpy as np
import pytest
import torch

from oracle import swimba_oracle as orc
from paper_2603_06938_amd import binding as sw
from paper_2603_06938_amd import synth
from gpu_util import IO, TOL, host, rel_errors

pytestmark = pytest.mark.gpu
SENTINEL = 7.0


def make_problem(B, L, Dm, E, G, N, io, seed):
    rng = np.random.default_rng(seed)
    rd = synth.round_to_bf16 if io == "bf16" else (lambda a: a)
    u = rd(rng.standard_normal((B, L, Dm)).astype(np.float32))
    # weights ~ N(0, 1/Dm): projected rows have unit-order entries
    WB = rd((rng.standard_normal((E, G, N, Dm)) / np.sqrt(Dm)).astype(np.float32))
    WC = rd((rng.standard_normal((E, G, N, Dm)) / np.sqrt(Dm)).astype(np.float32))
    g = rd(rng.standard_normal((B, L, E)).astype(np.float32))
    return u, WB, WC, g


def dev(a, io):
    return torch.from_numpy(np.ascontiguousarray(a)).to(IO[io]).to("cuda:0")


SHAPES = [
    # B, L, Dm, E, G, N, k, io
    (2, 37, 24, 4, 2, 8, 2, "f32"),
    (1, 50, 33, 5, 1, 20, 5, "f32"),        # dense routing, odd sizes
    (2, 40, 48, 4, 1, 24, 2, "bf16"),       # bf16 on the plain-arithmetic kernel (G*N % 64 != 0)
    (2, 300, 256, 8, 1, 128, 2, "bf16"),    # MFMA: ragged token tiles
    (1, 130, 80, 8, 2, 64, 1, "bf16"),      # MFMA: d_model = 64 + 16 (tail k-step), top-1
    (1, 70, 64, 16, 8, 128, 3, "bf16"),     # MFMA: 2048 output columns (8 column blocks), k = 3
    (1, 5, 32, 16, 1, 64, 2, "bf16"),       # MFMA: most experts receive no token
    (1, 256, 768, 8, 1, 128, 2, "bf16"),    # MFMA: a 130M-sized model width
    (1, 6200, 144, 1, 8, 128, 1, "bf16"),   # MFMA: one pass of 8 tiles a workgroup
    (1, 9001, 80, 2, 8, 128, 1, "bf16"),    # MFMA: passes of 5 tiles, two a workgroup
    (1, 12000, 32, 1, 8, 128, 1, "bf16"),   # MFMA: the same in less than one stage of features
    (1, 600, 64, 64, 8, 128, 2, "bf16"),    # MFMA: more experts than workgroups at once, lists in one piece
    (1, 66001, 32, 3, 1, 64, 2, "bf16"),    # MFMA: segments of the lists of more than 256 tokens
    (1, 300, 32, 32, 1, 64, 1, "bf16"),     # MFMA: most experts with segments, the second nearly empty
    (1, 300, 32, 32, 1, 64, 16, "bf16"),    # MFMA: and most slots: the routing takes more than 64 KB of LDS
]


@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: "B%dL%dD%dE%dG%dN%dk%d%s" % c)
def test_expert_proj_matches_oracle(cfg):
    B, L, Dm, E, G, N, k, io = cfg
    u, WB, WC, g = make_problem(B, L, Dm, E, G, N, io, seed=hash(cfg[:7]) % 100000)
    ref = orc.expert_proj(u, WB, WC, g, k, fill=SENTINEL)
    Bo = torch.full((B, L, E, G, N), SENTINEL, dtype=IO[io], device="cuda:0")
    Co = torch.full((B, L, E, G, N), SENTINEL, dtype=IO[io], device="cuda:0")
    out = sw.swimba_expert_proj(dev(u, io), dev(WB, io), dev(WC, io), dev(g, io), k, B_experts=Bo, C_experts=Co,
                                want_topk=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.topk_idx.cpu().numpy(), ref["topk_idx"])
    np.testing.assert_allclose(host(out.topk_w), ref["topk_w"], rtol=1e-5, atol=1e-30)
    keep = np.zeros((B, L, E), dtype=bool)
    np.put_along_axis(keep, ref["topk_idx"].astype(np.int64), True, axis=-1)
    for name, got, want in (("B", host(out.B_experts), ref["B_experts"]), ("C", host(out.C_experts), ref["C_experts"])):
        # rows of inactive experts are untouched
        assert (got[~keep] == SENTINEL).all(), name
        l2 = np.linalg.norm(got[keep] - want[keep]) / np.linalg.norm(want[keep])
        linf = np.abs(got[keep] - want[keep]).max() / np.abs(want[keep]).max()
        print(cfg, name, "rel l2 %.3e linf %.3e" % (l2, linf), flush=True)
        assert l2 <= TOL[io] and linf <= TOL[io], (name, l2, linf)


ROUTER_LINEAR_SHAPES = [
    # B, L, Dm, E, io
    (2, 37, 24, 4, "f32"), (1, 50, 33, 5, "f32"), (1, 3, 700, 256, "f32"),
    (2, 40, 48, 4, "bf16"), (1, 130, 77, 8, "bf16"),          # 77 features: element-wise path
    (2, 300, 768, 8, "bf16"), (1, 9, 1024, 16, "bf16"), (1, 1, 8, 1, "bf16"),
    # both sides of each width that a lane keeps in one, two and four pieces, and past it: piece ends inside the row and at its
    # end, last tokens and last experts that fill no wave
    (1, 7, 512, 9, "bf16"), (1, 6, 520, 8, "bf16"), (1, 5, 1032, 3, "bf16"), (2, 37, 1536, 8, "bf16"), (1, 33, 2048, 12, "bf16"),
    (1, 10, 2056, 8, "bf16"), (1, 3, 4096, 17, "bf16"),
]


@pytest.mark.parametrize("cfg", ROUTER_LINEAR_SHAPES, ids=lambda c: "B%dL%dD%dE%d%s" % c)
def test_router_linear_matches_oracle(cfg):
    B, L, Dm, E, io = cfg
    rng = np.random.default_rng(hash(cfg[:4]) % 100000)
    rd = synth.round_to_bf16 if io == "bf16" else (lambda a: a)
    u = rd(rng.standard_normal((B, L, Dm)).astype(np.float32))
    Wg = rd((rng.standard_normal((E, Dm)) / np.sqrt(Dm)).astype(np.float32))
    ref = orc.router_linear(u, Wg)
    got = sw.swimba_router_linear(dev(u, io), dev(Wg, io))
    torch.cuda.synchronize()
    assert got.shape == (B, L, E) and got.dtype == IO[io]
    g = host(got)
    l2 = np.linalg.norm(g - ref) / np.linalg.norm(ref)
    linf = np.abs(g - ref).max() / np.abs(ref).max()
    print(cfg, "logits rel l2 %.3e linf %.3e" % (l2, linf), flush=True)
    assert l2 <= TOL[io] and linf <= TOL[io], (l2, linf)


def test_projection_then_mixer_end_to_end():
    """Token features -> routed projection -> mixer, all on the GPU, against the oracle chain
    (oracle projections are not rounded to bf16 in between)."""
    B, L, Dm, E, G, N, k, H, P, Q = 2, 300, 128, 8, 1, 128, 2, 4, 64, 128
    u, WB, WC, g = make_problem(B, L, Dm, E, G, N, "bf16", seed=99)
    w = synth.Workload("e2e", B, L, H, P, N, G, E, k, Q, "bf16", 7)
    p = synth.make_inputs(w, seed=98)
    proj = sw.swimba_expert_proj(dev(u, "bf16"), dev(WB, "bf16"), dev(WC, "bf16"), dev(g, "bf16"), k)
    out = sw.swimba_mixer_fwd(dev(p["x"], "bf16"), dev(p["dt"], "bf16"), torch.from_numpy(p["A"]).to("cuda:0"), None,
                              proj.B_experts, proj.C_experts, dev(g, "bf16"), k, Q)
    torch.cuda.synchronize()
    rp = orc.expert_proj(u, WB, WC, g, k, fill=0.0)
    ref = orc.mixer_fwd(p["x"], p["dt"], p["A"], None, rp["B_experts"].astype(np.float32),
                        rp["C_experts"].astype(np.float32), g, k)
    l2, linf = rel_errors(host(out.y), ref["y"], (0, 2))
    print("projection + mixer: y rel l2 %.3e linf %.3e" % (l2, linf), flush=True)
    assert l2 <= TOL["bf16"] and linf <= TOL["bf16"], (l2, linf)


def test_expert_proj_empty_and_errors():
    d = "cuda:0"
    out = sw.swimba_expert_proj(torch.zeros((2, 0, 16), device=d), torch.zeros((3, 1, 4, 16), device=d),
                                torch.zeros((3, 1, 4, 16), device=d), torch.zeros((2, 0, 3), device=d), 2)
    assert out.B_experts.shape == (2, 0, 3, 1, 4)
    with pytest.raises(RuntimeError):
        sw.swimba_expert_proj(torch.zeros((1, 4, 16), device=d), torch.zeros((3, 1, 4, 16), device=d),
                              torch.zeros((3, 1, 4, 16), device=d), torch.zeros((1, 4, 3), device=d), 2,
                              workspace=torch.empty(256, dtype=torch.uint8, device=d))


@pytest.mark.parametrize("T,Dm,E,k,skew", [
    (257, 64, 8, 2, 0.0),          # one row tile a share and less
    (16384, 16, 4, 2, 0.0),        # four row tiles a share, one short stage
    (16385, 144, 8, 2, 0.0),       # and five; an odd number of stages
    (20000, 64, 4, 2, 0.0),        # shares of five to six row tiles
    (28000, 80, 4, 2, 0.0),        # of seven to eight
    (40000, 64, 16, 2, 3.0),       # of more than one pass, experts with few entries or none
    (70000, 32, 5, 1, 8.0),        # half a stage, most entries with one expert
])
def test_expert_proj_shares_and_passes(T, Dm, E, k, skew):
    """Every selected row of the grouped product, where the shares, their passes or the stages have their edges."""
    gen = torch.Generator(device="cuda:0").manual_seed(T)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda:0")
    u = rnd(1, T, Dm).bfloat16()
    WB, WC = [(rnd(E, 1, 64, Dm) * Dm ** -0.5).bfloat16() for _ in range(2)]
    logits = (rnd(1, T, E) - skew * torch.arange(E, device="cuda:0")).bfloat16()
    got = sw.swimba_expert_proj_selected(u, WB, WC, logits, k)
    idx = got.topk_idx.long()
    # the router's rule: logits descending, ties by the lower index
    order = torch.sort(logits.float(), dim=-1, descending=True, stable=True).indices[..., :k]
    assert torch.equal(idx, order)
    for out, W in ((got.B_experts, WB), (got.C_experts, WC)):
        want = torch.empty(T, k, 64, device="cuda:0")
        for e in range(E):
            rows = (idx[0] == e).nonzero(as_tuple=True)
            want[rows] = u[0, rows[0]].float() @ W[e, 0].float().T
        # half a unit in the last place of the bf16 result; fp32 sums in another order
        tol = 2.0 ** -8 * want.abs() + 1e-5 * Dm ** 0.5
        assert bool(((out[0, :, :, 0].float() - want).abs() <= tol).all())


@pytest.mark.parametrize("T,k,bad", [
    (257, 3, [3, 5] + [float("nan")] * 6),              # its pick by itself would repeat expert 1; a block of one token, the last one
    (257, 4, [9, float("nan"), 3, 5]),                  # the last expert, whose list ends the workspace
    (600, 4, [9] + [float("nan")] * 38 + [5]),          # lists in one piece
], ids=["E8", "E4", "E40"])
def test_a_token_without_an_order_leaves_the_others_alone(T, k, bad):
    """Logits that are NaN give unspecified picks, but distinct ones: the other tokens' rows and what lies behind the workspace
    stay as they are."""
    E, Dm = len(bad), 32
    gen = torch.Generator(device="cuda:0").manual_seed(T + E)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda:0")
    u = rnd(1, T, Dm).bfloat16()
    WB, WC = [(rnd(E, 1, 64, Dm) * Dm ** -0.5).bfloat16() for _ in range(2)]
    logits = rnd(1, T, E).bfloat16()
    logits[..., 1] += 8                              # an expert of every token: its list is full
    logits[..., E - 1] += 8
    size = sw.swimba_expert_proj_workspace_bytes(sw.make_dims(1, T, 1, 1, 64, 1, E, k, 1, torch.bfloat16), Dm)
    ws = torch.full((size + 4096,), 171, dtype=torch.uint8, device="cuda:0")
    want = sw.swimba_expert_proj_selected(u, WB, WC, logits, k)
    logits[0, T - 1] = torch.tensor(bad)
    got = sw.swimba_expert_proj_selected(u, WB, WC, logits, k, workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws[size:] == 171).all())
    for a, b in ((got.topk_idx, want.topk_idx), (got.B_experts, want.B_experts), (got.C_experts, want.C_experts)):
        assert torch.equal(a[:, :-1], b[:, :-1])
    picks = got.topk_idx[0, -1].sort().values
    assert 0 <= int(picks[0]) and int(picks[-1]) < E and bool((picks.diff() > 0).all())
