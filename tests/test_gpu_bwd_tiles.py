"""The backward's kernels where their tiles can go wrong: one to three chunks and the chunks around a checkpoint, whole and short, every
pair of head sizes and every gate layout, against the oracle; and the surplus rows of a short chunk's window, which
must reach nothing, whatever they hold."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2507_01004_amd import synth, zeco
from tests.gpu_util import TOL, checkpoints_only, host, rel_err_bh

pytestmark = pytest.mark.gpu
TOLB = TOL["bf16"]   # bf16 operands, fp32 accumulation: the bound of every bf16 test


def make(H, L, dk, dv, gate, seed, B=1):
    inp = synth.make_inputs(B, L, H, dk, dv, seed=seed, io="bf16", g="bf16" if gate == "bf16" else "f32", device="cuda",
                            per_head_gate=gate == "head", gate_div=64.0 if gate == "head" else 16.0)
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    inp["dO"] = torch.randn(inp["v"].shape, generator=gen, device="cuda").to(torch.bfloat16)
    return inp


@pytest.mark.parametrize("gate", ["f32", "bf16", "head"])
@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("L", [64, 65, 191, 192, 513, 640])
def test_gradients_of_one_segment(L, dk, dv, gate):
    inp = make(2, L, dk, dv, gate, 300 + L)
    h = {n: host(t) for n, t in inp.items()}
    if gate == "head":
        h["g"] = np.repeat(h["g"][..., None], dk, axis=-1)
    q, k, v, g, dO = (inp[n] for n in ("q", "k", "v", "g", "dO"))
    zero = torch.zeros(1, 1, 2, dk, dv, device="cuda")
    S, G = zeco.gla_local_state(k, v, g, 1)
    whole = zeco.gla_bwd_from_state(q, k, v, g, dO, zero, S[0], zero, 1, scale=0.5, workspace=checkpoints_only(q, v, g, 1)[0])
    cut = zeco.gla_bwd_from_state(q, k, v, g, dO, zero, S[0], zero, 1, scale=0.5)   # (from 512 tokens on)
    torch.cuda.synchronize()
    ref = oracle.gla_recurrent_bwd(h["q"], h["k"], h["v"], h["g"], h["dO"], 0.5, None, None)
    rg = ref[3].sum(axis=-1) if gate == "head" else ref[3]
    for got in (whole, cut):
        for nm, x, r in zip(("dq", "dk", "dv"), got[:3], ref[:3]):
            assert rel_err_bh(host(x), r, (0, 2)) <= TOLB, nm
        assert rel_err_bh(host(got[3]), rg, (0, 2)) <= TOLB, "dg"


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("dk,dv", [(64, 128), (128, 64), (128, 128)])
def test_surplus_rows_reach_nothing(dk, dv, bad):
    # 100 tokens: the reverse pass loads the last 36 as the window [36, 100), whose first 28 rows belong to the chunk before
    inp = make(1, 100, dk, dv, "f32", 900 + dk)
    q, k, v, g, dO = (inp[n] for n in ("q", "k", "v", "g", "dO"))
    zero = torch.zeros(1, 1, 1, dk, dv, device="cuda")
    S, _ = zeco.gla_local_state(k, v, g, 1)
    clean = zeco.gla_bwd_from_state(q, k, v, g, dO, zero, S[0], zero, 1)
    dO2 = dO.clone()
    dO2[:, 40] = bad
    got = zeco.gla_bwd_from_state(q, k, v, g, dO2, zero, S[0], zero, 1)
    torch.cuda.synchronize()
    assert torch.equal(got[0][:, :40], clean[0][:, :40]) and torch.equal(got[0][:, 41:], clean[0][:, 41:])
    for a, b in zip(got[1:], clean[1:]):   # what depends on later tokens only
        assert torch.equal(a[:, 64:], b[:, 64:])


@pytest.mark.parametrize("gate", ["f32", "bf16", "head"])
@pytest.mark.parametrize("dv", [64, 128])
@pytest.mark.parametrize("streams", [64, 65, 128, 129])
def test_state_passes_and_dq_around_the_sibling_rules(streams, dv, gate):
    # 64 and 128 streams are the last that run as four and as two workgroups a stream (state passes; dQ: two)
    P, L, dk = streams, 96, 128
    inp = make(1, P * L, dk, dv, gate, 40 + streams)
    h = {n: host(t) for n, t in inp.items()}
    if gate == "head":
        h["g"] = np.repeat(h["g"][..., None], dk, axis=-1)
    q, k, v, g, dO = (inp[n] for n in ("q", "k", "v", "g", "dO"))
    S_loc, G_tot = zeco.gla_local_state(k, v, g, P)
    S_init, S_last = zeco.state_scan(S_loc, G_tot)
    dS_loc = zeco.gla_bwd_dstate(q, g, dO, P, scale=0.5)
    dS_in, dS0 = zeco.state_scan(dS_loc, G_tot, direction=1)
    got = zeco.gla_bwd_from_state(q, k, v, g, dO, S_init, S_last, dS_in, P, scale=0.5)
    torch.cuda.synchronize()
    _, S_ref = oracle.gla_recurrent(h["q"], h["k"], h["v"], h["g"], 0.5)
    ref = oracle.gla_recurrent_bwd(h["q"], h["k"], h["v"], h["g"], h["dO"], 0.5, None, None)
    assert rel_err_bh(host(S_last), S_ref, (0, 1)) <= TOLB
    assert rel_err_bh(host(dS0), ref[4], (0, 1)) <= TOLB
    assert rel_err_bh(host(G_tot).sum(axis=0)[..., None], h["g"][..., 0].sum(axis=1)[..., None] if gate == "head" else h["g"].sum(axis=1)[..., None],
                      (0, 1)) <= 1e-5
    for nm, x, r in zip(("dq", "dk", "dv"), got[:3], ref[:3]):
        assert rel_err_bh(host(x), r, (0, 2)) <= TOLB, nm
    assert rel_err_bh(host(got[3]), ref[3].sum(axis=-1) if gate == "head" else ref[3], (0, 2)) <= TOLB, "dg"


def check_batch(inp, gate, got, samples, scale):
    """Gradients (and the initial state's, if given) of a few batch entries of one segment each, against the oracle."""
    for b in samples:
        h = {n: host(t[b:b + 1]) for n, t in inp.items()}
        if gate == "head":
            h["g"] = np.repeat(h["g"][..., None], h["q"].shape[-1], axis=-1)
        ref = list(oracle.gla_recurrent_bwd(h["q"], h["k"], h["v"], h["g"], h["dO"], scale, None, None))
        if gate == "head":
            ref[3] = ref[3].sum(axis=-1)
        for nm, x, r in zip(("dq", "dk", "dv", "dg", "dS0"), got, ref):
            assert rel_err_bh(host(x[b:b + 1]), r, (0, 1) if nm == "dS0" else (0, 2)) <= TOLB, (nm, b)


def from_state(inp, L, dk, dv, scale):
    B, H = inp["q"].shape[0], inp["q"].shape[2]
    zero = torch.zeros(1, B, H, dk, dv, device="cuda")
    S, _ = zeco.gla_local_state(inp["k"], inp["v"], inp["g"], 1)
    return zeco.gla_bwd_from_state(*(inp[n] for n in ("q", "k", "v", "g", "dO")), zero, S[0], zero, 1, scale=scale,
                                   workspace=checkpoints_only(inp["q"], inp["v"], inp["g"], 1)[0])   # (whole segments)


@pytest.mark.parametrize("gate", ["f32", "bf16", "head"])
@pytest.mark.parametrize("dv", [64, 128])
@pytest.mark.parametrize("L", [513, 640])
def test_more_streams_than_siblings_take_with_checkpoints(L, dv, gate):
    """130 streams: one workgroup each in the dQ pass too, with a checkpoint behind the eighth chunk and a short or whole last one."""
    inp = make(1, L, 128, dv, gate, 510 + L, B=130)
    got = from_state(inp, L, 128, dv, 0.5)
    torch.cuda.synchronize()
    check_batch(inp, gate, got, (0, 64, 129), 0.5)


@pytest.mark.parametrize("B,dk,dv,gate", [
    (130, 128, 128, "f32"), (130, 128, 128, "bf16"), (130, 128, 128, "head"),
    (130, 64, 64, "f32"), (130, 64, 64, "bf16"), (130, 64, 64, "head"),
    (130, 64, 128, "f32"), (130, 64, 128, "bf16"), (130, 64, 128, "head"),
    (130, 128, 64, "f32"), (130, 128, 64, "bf16"), (130, 128, 64, "head"),
    (100, 128, 128, "bf16"), (100, 128, 64, "f32"),          # dQ pass of from_state in siblings
])
def test_gradients_past_the_caches(B, dk, dv, gate):
    """Tensors of over 215e6 bytes (q, k, v, dO and the gates) take the kernels with non-temporal rows; the length leaves a short chunk."""
    per_token = 4 * (dk + dv) + {"f32": 4 * dk, "bf16": 2 * dk, "head": 4}[gate]
    L = int(215e6 / (B * per_token)) + 8
    L += 1 - L % 2
    assert B * L * per_token > 215e6 and L % 64
    inp = make(1, L, dk, dv, gate, 70 + B + dv, B=B)
    q, k, v, g, dO = (inp[n] for n in ("q", "k", "v", "g", "dO"))
    got = from_state(inp, L, dk, dv, 0.5)
    fused = zeco.gla_fused_bwd(q, k, v, g, dO, 1, scale=0.5)
    torch.cuda.synchronize()
    check_batch(inp, gate, got, (0, B - 1), 0.5)
    check_batch(inp, gate, fused, (0, B - 1), 0.5)
