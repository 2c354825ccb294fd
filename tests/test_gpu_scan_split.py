"""The scan of a long chain of few elements, split over the waves of a workgroup: against the recurrence in 64 bits at the edges of its
runs (32 segments), its rounds (256) and its rule, in both directions, for both gate layouts and with chains in groups."""
import pytest
import torch

from paper_2507_01004_amd import synth, zeco
from tests.gpu_util import host, randn_seeded, rel_err_bh

pytestmark = pytest.mark.gpu

# (P, BH, d_k, d_v, per-head gates, direction, S0)
CASES = [(24, 1, 64, 64, False, 0, True), (32, 4, 128, 128, False, 1, False), (25, 2, 64, 128, True, 1, False), (256, 1, 128, 128, False, 0, True), (257, 1, 64, 64, True, 0, False),
         (31, 4, 128, 64, False, 1, True), (511, 3, 64, 64, False, 1, True), (160, 4, 128, 128, False, 0, True), (161, 4, 128, 128, False, 0, True),
         (1025, 1, 128, 64, False, 0, True)]


def _inputs(P, BH, dk, dv, head, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    S = torch.randn(P, 1, BH, dk, dv, generator=gen, device="cuda")
    G = -0.5 * torch.rand((P, 1, BH) if head else (P, 1, BH, dk), generator=gen, device="cuda")
    return S, G, torch.randn(1, BH, dk, dv, generator=gen, device="cuda")


def _exact(S, G, S0, head, reverse):
    s = torch.zeros(S.shape[1:], dtype=torch.float64, device="cuda") if S0 is None else S0.double()
    out = torch.empty(S.shape, dtype=torch.float64, device="cuda")
    for p in (reversed(range(S.shape[0])) if reverse else range(S.shape[0])):
        out[p] = s
        s = s * (G[p].double().exp()[..., None, None] if head else G[p].double().exp()[..., None]) + S[p].double()
    return out, s


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_scan_is_the_recurrence(case):
    P, BH, dk, dv, head, reverse, with_s0 = case
    print("case", case, flush=True)
    S, G, S0 = _inputs(P, BH, dk, dv, head, P)
    S0 = S0 if with_s0 else None
    got, last = zeco.state_scan(S, G, S0=S0, direction=reverse)
    again, last2 = zeco.state_scan(S, G, S0=S0, direction=reverse, K_blocks=1)
    ref, ref_last = _exact(S, G, S0, head, reverse)
    torch.cuda.synchronize()
    assert torch.equal(got, again) and torch.equal(last, last2)            # repeatable, whatever the row blocks
    first = got[P - 1 if reverse else 0]
    assert torch.equal(first, S0 if with_s0 else torch.zeros_like(first))   # what enters the chain enters its first segment
    # decays of 0.78 on average: some five steps of 2^-24 each, and the decays' own 2^-22, in the size of a state (2-norms)
    for x, r in ((got, ref), (last, ref_last)):
        assert ((x - r).norm() / r.norm()).item() <= 3e-7
        assert ((x - r).abs().max() / r.abs().max()).item() <= 2e-6


def test_what_is_no_number_stays_behind_its_segment():
    S, G, S0 = _inputs(300, 1, 64, 64, False, 7)
    S[70, 0, 0, 3, 5] = float("nan")
    S[290, 0, 0, 9, 9] = float("inf")
    got, last = zeco.state_scan(S, G, S0=S0)
    torch.cuda.synchronize()
    assert torch.isfinite(got[:71]).all() and torch.isnan(got[71:, 0, 0, 3, 5]).all()
    bad = ~torch.isfinite(got)
    bad[:, 0, 0, 3, 5] = False
    bad[:, 0, 0, 9, 9] = False
    assert not bad.any() and torch.isfinite(got[:291, 0, 0, 9, 9]).all() and not torch.isfinite(last[0, 0, 9, 9])


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (128, 128)])
def test_one_head_in_512_pieces_either_side_of_the_trees_rule(dk, dv):
    """The one-call forms in fp32 over one head of 131072 tokens: 512 pieces, scanned as a tree up to 8192 elements a state and as one chain
    beyond; against the same head twice, which is never scanned as a tree.  (Sums in another order: 1e-5, dg, whose terms cancel, 1e-4.)"""
    T = 131072
    print("512 pieces", dk, dv, flush=True)
    inp = synth.make_inputs(1, T, 1, dk, dv, seed=dk + dv, io="f32", g="f32", device="cuda", gate_div=64.0)
    one = [inp[n] for n in "qkvg"] + [randn_seeded(tuple(inp["v"].shape), 81)]
    two = [x.expand(1, T, 2, x.shape[-1]).contiguous() for x in one]
    S0, dS_T = (0.3 * randn_seeded((1, 1, dk, dv), i) for i in (82, 83))
    rest = zeco.fused_workspace_bytes(one[0], one[2], one[3], 1) - 4 * 512 * (2 * dk * dv + 4 * dk)   # states and decays of 512 pieces
    tree = zeco.lib().zeco_state_scan_tree_workspace(512, 1, dk, dv, 0)
    assert rest >= tree if dk * dv <= 8192 else 0 <= rest < tree
    out = []
    for x, s0, ds in ((one, S0, dS_T), (two, S0.repeat(1, 2, 1, 1), dS_T.repeat(1, 2, 1, 1))):
        q, k, v, g, dO = x
        o, S = zeco.gla_fused_fwd(q, k, v, g, 1, S0=s0)
        out.append((o, S) + tuple(zeco.gla_fused_bwd(q, k, v, g, dO, 1, S0=s0, dS_T=ds)))
    torch.cuda.synchronize()
    for i, (x, y) in enumerate(zip(*out)):
        y = y[:, :1] if x.shape[1] == 1 else y[:, :, :1]   # states, token rows
        assert rel_err_bh(host(x), host(y), (0,)) <= (1e-4 if i == 5 else 1e-5), i
