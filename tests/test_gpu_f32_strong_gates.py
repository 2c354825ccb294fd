"""fp32 results over the whole range of gates: the sum of |g| over a chunk may come close to 160, in whatever tokens, with operands of
any ordinary size.  The decay of a 32-token window then spans e^-158, more than the parts of a split operand can carry, so these
cases are where the kernels at C = 32 and 64 have to take the fp32 instructions; everything is held against the chunk-free
recurrence in 64 bits at the fp32 tolerance (2e-5 of it is what rounding a cumulative log decay of 160 to fp32, 2^-17, leaves twice)."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2507_01004_amd import synth, zeco
from tests.gpu_util import TOL, host, randn_seeded, rel_err_bh

pytestmark = pytest.mark.gpu


def _inputs(C, total, where, size, T, dk, dv, B=1, H=2):
    """Normal q, v and dO, unit k; `total` of log decay in every C tokens: all of it in one token, a different one per channel
    ("token"), in C's first eight ("front"), or in one token of every third chunk only ("rare")."""
    inp = synth.make_inputs(B, T, H, dk, dv, seed=int(10 * total) + C + dk, io="f32", g="f32", device="cuda", gate_div=64.0)
    q, k, v = (inp[n] for n in "qkv")
    dO = randn_seeded(tuple(v.shape), 41)
    gen = torch.Generator(device="cuda").manual_seed(42)
    g = -1e-3 * torch.rand(q.shape, generator=gen, device="cuda")
    # (the same place in every chunk, so that no window of C tokens, wherever the chunks begin, holds more than `total`)
    at = torch.randint(0, C, (H, dk), generator=gen, device="cuda")
    for i, a in enumerate(range(0, T, C)):
        if where == "front":
            g[:, a:a + 8] -= total / 8
        elif where == "token" or i % 3 == 1:
            t = torch.arange(a, min(a + C, T), device="cuda")
            g[:, a:a + C] -= total * (t[:, None, None] - a == at)
    if size == "kv":        # rows whose products with a factor of e^79 pass the largest fp32 value, with results of ordinary size
        return q, k * 100, v * 100, g, dO * 0.01
    if size == "qdo":
        return q * 30, k, v * 0.003, g, dO * 300
    return q * size, k, v, g, dO * size


@pytest.mark.parametrize("size", [1.0, 1e-3, 1e-6, "kv", "qdo"])
@pytest.mark.parametrize("case", [(64, 158.0, "token", 256, 128, 128), (32, 158.0, "front", 256, 128, 128), (32, 140.0, "token", 225, 64, 64),
                                  (32, 126.0, "front", 97, 64, 128), (32, 158.0, "rare", 321, 128, 64), (64, 100.0, "token", 130, 64, 64)],
                         ids=lambda c: "C%d_%d_%s_T%d_%dx%d" % c)
def test_results_are_fp32_over_the_range_of_gates(case, size):
    C, total, where, T, dk, dv = case
    print("case", case, size, flush=True)
    q, k, v, g, dO = _inputs(C, total, where, size, T, dk, dv)
    B, H = q.shape[0], q.shape[2]
    S0 = 0.3 * randn_seeded((B, H, dk, dv), 44)
    dS_T = 0.3 * randn_seeded((B, H, dk, dv), 45) * (size if size in (1.0, 1e-3, 1e-6) else 1.0)
    o, S = zeco.gla_fused_fwd(q, k, v, g, 1, S0=S0, C=C)
    S_loc, _ = zeco.gla_local_state(k, v, g, 1, C=C)
    o_s = zeco.gla_fwd_from_state(q, k, v, g, S0[None], 1, C=C)
    dS_loc = zeco.gla_bwd_dstate(q, g, dO, 1, C=C)
    got = zeco.gla_fused_bwd(q, k, v, g, dO, 1, S0=S0, dS_T=dS_T, C=C)
    torch.cuda.synchronize()
    h = [host(x) for x in (q, k, v, g)]
    o_r, S_r = oracle.gla_recurrent(*h, 1.0, host(S0))
    _, S_z = oracle.gla_recurrent(*h, 1.0, None)
    ref = oracle.gla_recurrent_bwd(*h, host(dO), 1.0, host(S0), host(dS_T))
    dS_z = oracle.gla_recurrent_bwd(*h, host(dO), 1.0, None, None)[4]
    pairs = [("o", o, o_r, (0, 2)), ("S", S, S_r, (0, 1)), ("S_loc", S_loc[0], S_z, (0, 1)), ("o_s", o_s, o_r, (0, 2)), ("dS_loc", dS_loc[0], dS_z, (0, 1)),
             ("dq", got[0], ref[0], (0, 2)), ("dk", got[1], ref[1], (0, 2)), ("dv", got[2], ref[2], (0, 2)),
             ("dS0", got[4], ref[4], (0, 1))]
    errs = {name: rel_err_bh(host(x), np.asarray(r), axes) for name, x, r, axes in pairs}
    # dg is a running sum of terms q dq and k dk that cancel (down to nothing where all that comes later has decayed): its rounding is theirs
    terms = np.maximum(np.abs(h[0] * ref[0]), np.abs(h[1] * ref[1])).max(axis=(1, 3), keepdims=True)
    errs["dg"] = float(np.max(np.abs(host(got[3]) - ref[3]) / np.maximum(terms, np.abs(ref[3]).max(axis=(1, 3), keepdims=True))))
    print(" ".join("%s %.1e" % e for e in errs.items()), flush=True)
    for name, err in errs.items():
        assert err <= TOL["f32"], name
