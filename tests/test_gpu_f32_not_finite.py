"""fp32 inputs that hold an infinity, a NaN or a value near the largest: at C = 32 and 64, where operands are split, the values spread as far
as on the fp32 instructions and no further - a column of v or dO stays a column of o, dv and the states, what comes before the
token's sixteen stays finite, and an infinity that meets numbers stays an infinity of its sign instead of a NaN."""
import pytest
import torch

from paper_2507_01004_amd import synth, zeco
from tests.gpu_util import randn_seeded

pytestmark = pytest.mark.gpu

INF, NAN, BIG = float("inf"), float("nan"), 3.4e38
B, T, H = 1, 256, 1


def _inputs(dk, dv):
    inp = synth.make_inputs(B, T, H, dk, dv, seed=dk + dv, io="f32", g="f32", device="cuda")
    q, k, v, g = (inp[n] for n in "qkvg")
    # (q and k positive, so that a product with an infinity has a sign wherever it is one)
    return q.abs() + 0.1, k.abs() + 0.01, v, g, randn_seeded(tuple(v.shape), 5)


def _tokens(x):
    """Tokens with a value that is not finite."""
    return (~torch.isfinite(x)).flatten(2).any(-1)[0].nonzero().flatten().tolist()


@pytest.mark.parametrize("C", [32, 64])
@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (64, 128), (128, 64)], ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("bad", [INF, -INF, NAN, BIG])
def test_a_value_of_v_stays_in_its_column(dims, bad, C):
    dk, dv = dims
    t0, j = 140, 7
    print("case", dims, bad, C, flush=True)
    q, k, v, g, dO = _inputs(dk, dv)
    v[0, t0, 0, j] = bad
    S_loc, _ = zeco.gla_local_state(k, v, g, 1, C=C)
    o, S = zeco.gla_fused_fwd(q, k, v, g, 1, C=C)
    o_s = zeco.gla_fwd_from_state(q, k, v, g, torch.zeros_like(S)[None], 1, C=C)
    torch.cuda.synchronize()
    cols = [c for c in range(dv) if c != j]
    for x in (o, o_s):
        assert torch.isfinite(x[..., cols]).all()
        assert all(t >= t0 // 16 * 16 for t in _tokens(x))
        if bad == bad:   # with a sign of its own from its token on
            assert (x[0, t0:t0 + 8, 0, j] == (bad if abs(bad) == INF else x[0, t0:t0 + 8, 0, j])).all() and not torch.isnan(x[0, t0:, 0, j]).any()
        else:
            assert torch.isnan(x[0, t0:, 0, j]).all()
    for x in (S_loc[0], S):
        assert torch.isfinite(x[..., cols]).all()
        assert torch.isnan(x[..., j]).all() if bad != bad else not torch.isnan(x[..., j]).any()


@pytest.mark.parametrize("dims", [(64, 64), (128, 128)], ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("bad", [INF, NAN, BIG])
def test_a_value_of_the_incoming_state_stays_in_its_column(dims, bad):
    dk, dv = dims
    print("case", dims, bad, flush=True)
    q, k, v, g, dO = _inputs(dk, dv)
    S0 = 0.3 * randn_seeded((1, B, H, dk, dv), 6)
    S0[0, 0, 0, 5, 9] = bad
    o = zeco.gla_fwd_from_state(q, k, v, g, S0, 1)
    torch.cuda.synchronize()
    cols = [c for c in range(dv) if c != 9]
    assert torch.isfinite(o[..., cols]).all()
    assert torch.isnan(o[..., 9]).all() if bad != bad else not torch.isnan(o[..., 9]).any() and (o[..., 9] > 1e30).all()


@pytest.mark.parametrize("C", [32, 64])
@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (64, 128), (128, 64)], ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("bad", [INF, NAN, BIG])
def test_gradients_keep_to_their_columns_and_tokens(dims, bad, C):
    """A value of dO reaches its column of dv and of the states' gradients, and no token behind its sixteen; dq of its own token only."""
    dk, dv = dims
    t0, j = 115, 11
    print("case", dims, bad, C, flush=True)
    q, k, v, g, dO = _inputs(dk, dv)
    dO[0, t0, 0, j] = bad
    dS = zeco.gla_bwd_dstate(q, g, dO, 1, C=C)[0]
    dq, dk_, dv_, dg, dS0 = zeco.gla_fused_bwd(q, k, v, g, dO, 1, C=C)
    torch.cuda.synchronize()
    cols = [c for c in range(dv) if c != j]
    for x in (dS, dS0, dv_):
        assert torch.isfinite(x[..., cols]).all()
        if bad == bad:
            assert not torch.isnan(x[..., j] if x.dim() == 4 and x is not dv_ else x[0, :t0, 0, j]).any()
    last = t0 // 16 * 16 + 15
    assert all(t <= last for t in _tokens(dv_)) and all(t <= last for t in _tokens(dk_))
    if bad != BIG:
        assert _tokens(dq) == [t0]
