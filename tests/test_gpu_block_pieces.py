"""The building blocks with a workspace: over few streams the library cuts every segment into pieces, and each call has to
give what the same call without a workspace gives - states, outputs and gradients per segment - over every layout, dtype,
chunk length and raggedness it takes, at counts of pieces that do and do not divide the segment."""
import ctypes

import pytest
import torch

from paper_2507_01004_amd import zeco
from tests.gpu_util import host, randn_seeded, rel_err_bh

# (B, H, P, L, d_k, d_v, gate, io, C, head-major storage, wide gates), the calls that are cut (0 states, 1 output pass, 2 state gradients,
# 3 gradients), pieces per segment and checkpoints of dG inside the longest of them in the gradient call (as its workspace has them)
CASES = [
    ((1, 1, 1, 512, 128, 128, "f32", "bf16", 64, False, False), "0123", 8, 0),     # one chunk a piece, the shortest segment that is cut
    ((2, 2, 3, 1000, 128, 128, "f32", "bf16", 64, False, False), "0123", 8, 0),    # ragged, pieces of two lengths, several batch entries
    ((1, 4, 4, 8191, 64, 128, "bf16", "bf16", 64, False, False), "0123", 16, 0),   # 63-token remainder
    ((1, 3, 2, 2048, 128, 64, "head", "bf16", 64, False, False), "0123", 32, 0),
    ((1, 8, 4, 1664, 64, 64, "f32", "bf16", 64, True, False), "0123", 8, 0),       # 26 chunks: pieces that do not come out even
    ((2, 16, 4, 4099, 128, 128, "f32", "bf16", 64, False, False), "03", 2, 4),     # 128 streams: two pieces a segment at most
    ((1, 16, 4, 5000, 128, 128, "f32", "bf16", 64, False, False), "0123", 4, 2),   # 256 pieces: whole streams, the last pieces left out
    ((1, 16, 8, 4001, 64, 64, "head", "bf16", 64, False, False), "023", 2, 3),
    ((1, 2, 2, 1100, 128, 128, "f32", "bf16", 64, False, True), "0123", 9, 0),     # twice the range of gates
    ((1, 2, 2, 1000, 128, 128, "f32", "f32", 64, False, False), "0123", 8, 0),
    ((1, 16, 4, 4200, 128, 128, "f32", "f32", 64, False, False), "0123", 8, 1),    # checkpoints inside unequal pieces
    ((1, 20, 5, 3000, 128, 64, "f32", "f32", 32, False, False), "0123", 5, 1),
    ((1, 3, 2, 777, 64, 128, "f32", "f32", 32, True, False), "0123", 8, 0),
    ((2, 1, 2, 530, 128, 64, "f32", "f32", 16, False, False), "0123", 8, 0),
]


def _inputs(case):
    B, H, P, L, dk, dv, gate, io, C, hm, wide = case
    T, dt = P * L, torch.bfloat16 if io == "bf16" else torch.float32

    def lay(x, dtype):   # [B,T,H,d], stored head-major or token-major
        return x.to(dtype).transpose(1, 2) if hm else x.to(dtype)

    q, k = (randn_seeded((B, H, T, dk) if hm else (B, T, H, dk), s) for s in (1, 2))
    v, dO = (randn_seeded((B, H, T, dv) if hm else (B, T, H, dv), s) for s in (3, 4))
    k = k / k.norm(dim=-1, keepdim=True)
    if gate == "head":
        g = torch.nn.functional.logsigmoid(randn_seeded((B, T, H), 5)) / 16
    else:
        g = torch.nn.functional.logsigmoid(randn_seeded(tuple(q.shape), 5)) / (4 if wide else 16)
        g = lay(g, torch.bfloat16 if gate == "bf16" else torch.float32)
    gd = () if gate == "head" else (dk,)
    return lay(q, dt), lay(k, dt), lay(v, dt), g, lay(dO, dt), gd


def _whole(desc, name, args):
    """The call without a workspace (zeco_gla_bwd_from_state: with that of its checkpoints alone)."""
    L = zeco.lib()
    ptrs = [x.data_ptr() for x in args]
    if name == "zeco_gla_bwd_from_state":
        need = L.zeco_gla_bwd_from_state_workspace(ctypes.byref(desc))
        ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        ptrs += [ws.data_ptr(), need]
        st = getattr(L, name)(ctypes.byref(desc), *ptrs, zeco._stream())
        torch.cuda.synchronize()
    else:
        st = getattr(L, name)(ctypes.byref(desc), *ptrs, zeco._stream())
    assert st == zeco.ZECO_OK


@pytest.mark.gpu
@pytest.mark.parametrize("case, cut, pieces, ck", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_cut_calls_give_what_whole_segments_give(case, cut, pieces, ck):
    B, H, P, L, dk, dv, gate, io, C, hm, wide = case
    print("block pieces", case, flush=True)
    q, k, v, g, dO, gd = _inputs(case)
    f32 = lambda *s: torch.empty(s, device="cuda")
    # whole and cut differ by the order of sums only: what the operand type leaves of a state passed on in fp32 once more
    # (bf16: 2^-9 a product; dg, whose terms cancel, the bound of its own tests)
    tol, tol_dg = (1e-2, 2e-2) if io == "bf16" else (1e-5, 1e-4)
    with zeco.wide_gates(wide):
        desc = zeco.make_desc(q, v, g, P, C, 0.5)
        sizes = [zeco.lib().zeco_gla_block_workspace(ctypes.byref(desc), c) for c in range(4)]
        whole = [0, 0, 0, zeco.lib().zeco_gla_bwd_from_state_workspace(ctypes.byref(desc))]
        assert "".join(str(c) for c in range(4) if sizes[c] > whole[c]) == cut
        assert sizes[3] == 4 * P * B * H * pieces * ((3 + ck) * dk * dv + 2 * dk)
        S_loc, G_tot = zeco.gla_local_state(k, v, g, P, C=C)
        S_w, G_w = f32(P, B, H, dk, dv), f32(P, B, H, *gd)
        _whole(desc, "zeco_gla_local_state", (k, v, g, S_w, G_w))
        S0 = 0.3 * randn_seeded((B, H, dk, dv), 6)
        S_init, S_last = zeco.state_scan(S_w, G_w, S0=S0)
        o = zeco.gla_fwd_from_state(q, k, v, g, S_init, P, scale=0.5, C=C)
        o_w = torch.empty_like(o)
        _whole(desc, "zeco_gla_fwd_from_state", (q, k, v, g, S_init, o_w))
        dS = zeco.gla_bwd_dstate(q, g, dO, P, scale=0.5, C=C)
        dS_w = torch.empty_like(dS)
        _whole(desc, "zeco_gla_bwd_dstate", (q, g, dO, dS_w))
        dS_in, _ = zeco.state_scan(dS_w, G_w, S0=0.3 * randn_seeded((B, H, dk, dv), 7), direction=1)
        grads = zeco.gla_bwd_from_state(q, k, v, g, dO, S_init, S_last, dS_in, P, scale=0.5, C=C)
        grads_w = tuple(torch.empty_like(x) for x in grads)
        _whole(desc, "zeco_gla_bwd_from_state", (q, k, v, g, dO, S_init, S_last, dS_in) + grads_w)
    torch.cuda.synchronize()
    # log decays: added up in 64 bits either way, so that they are rounded once (the fp32 kernel and per-channel gates: equal)
    assert torch.allclose(G_tot, G_w, rtol=2e-7, atol=1e-6)
    for name, x, ref, axes, t in (("S_loc", S_loc, S_w, (0, 1, 2), tol), ("o", o, o_w, (0, 2), tol),
                                  ("dS_loc", dS, dS_w, (0, 1, 2), tol), ("dq", grads[0], grads_w[0], (0, 2), tol),
                                  ("dk", grads[1], grads_w[1], (0, 2), tol), ("dv", grads[2], grads_w[2], (0, 2), tol),
                                  ("dg", grads[3], grads_w[3], (0, 2), tol_dg)):
        assert rel_err_bh(host(x), host(ref), axes) <= t, name


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_the_call_without_leave_to_cut_keeps_to_its_own_size(io):
    """zeco_gla_bwd_from_state with more workspace than it asks for: the same bits as with exactly that, and not a byte past it."""
    case = (1, 2, 2, 2048, 128, 128, "f32", io, 64, False, False)
    B, H, P, L, dk, dv = case[:6]
    print("arena", io, flush=True)
    q, k, v, g, dO, gd = _inputs(case)
    desc = zeco.make_desc(q, v, g, P, 64, 0.5)
    need = zeco.lib().zeco_gla_bwd_from_state_workspace(ctypes.byref(desc))
    more = zeco.lib().zeco_gla_block_workspace(ctypes.byref(desc), zeco.BLOCK_BWD_FROM_STATE)
    assert 0 < need < more
    S, S_last, dS = (0.3 * randn_seeded(s, i) for i, s in enumerate([(P, B, H, dk, dv), (B, H, dk, dv), (P, B, H, dk, dv)], 50))
    arena = torch.full((more + 4096,), 171, dtype=torch.uint8, device="cuda")
    out = []
    for ws in (torch.empty(need, dtype=torch.uint8, device="cuda"), arena):
        grads = tuple(torch.empty_like(x) for x in (q, k, v)) + (torch.empty(g.shape, device="cuda"),)
        st = zeco.lib().zeco_gla_bwd_from_state(ctypes.byref(desc), *[x.data_ptr() for x in (q, k, v, g, dO, S, S_last, dS) + grads + (ws,)],
                                                ws.numel(), zeco._stream())
        assert st == zeco.ZECO_OK
        out.append(grads)
    by_binding = zeco.gla_bwd_from_state(q, k, v, g, dO, S, S_last, dS, P, scale=0.5, workspace=arena)
    torch.cuda.synchronize()
    assert (arena[need:] == 171).all()
    for x, y, z in zip(*out, by_binding):
        assert torch.equal(x, y) and torch.equal(x, z)


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_a_workspace_of_the_programs_own(io, monkeypatch):
    """The binding's `block_workspace`: with one of the size asked for the bits are those of a call that takes it from the pool, and nothing
    is allocated; with an empty one, and where the pool has no room, they are those of whole segments."""
    case = (1, 2, 2, 2048, 128, 64, "f32", io, 64, False, False)
    B, H, P, L, dk, dv = case[:6]
    print("kept workspace", io, flush=True)
    q, k, v, g, dO, gd = _inputs(case)
    f32 = lambda *s: torch.empty(s, device="cuda")
    S, S_last, dS = (0.3 * randn_seeded(s, i) for i, s in enumerate([(P, B, H, dk, dv), (B, H, dk, dv), (P, B, H, dk, dv)], 60))
    outs = lambda: (f32(P, B, H, dk, dv), f32(P, B, H, *gd), torch.empty_like(v), f32(P, B, H, dk, dv),
                    (torch.empty_like(q), torch.empty_like(k), torch.empty_like(v), f32(*g.shape)))

    def run(out, ws):
        zeco.gla_local_state(k, v, g, P, out=out[:2], block_workspace=ws[0])
        zeco.gla_fwd_from_state(q, k, v, g, S, P, scale=0.5, out=out[2], block_workspace=ws[1])
        zeco.gla_bwd_dstate(q, g, dO, P, scale=0.5, out=out[3], block_workspace=ws[2])
        zeco.gla_bwd_from_state(q, k, v, g, dO, S, S_last, dS, P, scale=0.5, out=out[4], block_workspace=ws[3])
        torch.cuda.synchronize()
        return out[:4] + out[4]

    sizes = [zeco.block_workspace_bytes(x, y, g, P, c) for c, (x, y) in enumerate([(k, v), (q, v), (q, dO), (q, v)])]
    assert all(n > 0 for n in sizes)
    kept = [torch.empty(n, dtype=torch.uint8, device="cuda") for n in sizes]
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    pool, whole = run(outs(), [None] * 4), run(outs(), [none] * 4)
    own, poor = outs(), outs()
    real = torch.empty

    def refuse(*a, **kw):
        raise AssertionError("allocated")

    def no_room(n, *a, **kw):
        if n in sizes:   # (the checkpoints of whole segments are another, smaller request)
            raise torch.cuda.OutOfMemoryError("no room")
        return real(n, *a, **kw)

    monkeypatch.setattr(torch, "empty", refuse)
    own = run(own, kept)
    monkeypatch.setattr(torch, "empty", no_room)
    poor = run(poor, [None] * 4)
    monkeypatch.setattr(torch, "empty", real)
    assert all(torch.equal(x, y) for x, y in zip(pool, own))
    assert all(torch.equal(x, y) for x, y in zip(whole, poor))
    assert not all(torch.equal(x, y) for x, y in zip(pool, whole))   # (cut and whole differ in the last bits: something was cut)


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_workspaces_the_calls_cannot_use(io):
    """The _ws forms with no workspace, one byte too few or a misaligned one: whole segments, as the calls without one run them."""
    case = (1, 2, 2, 2048, 128, 128, "f32", io, 64, False, False)
    B, H, P, L, dk, dv = case[:6]
    print("unusable workspaces", io, flush=True)
    q, k, v, g, dO, gd = _inputs(case)
    f32 = lambda *s: torch.empty(s, device="cuda")
    S, S_last, dS = (0.3 * randn_seeded(s, i) for i, s in enumerate([(P, B, H, dk, dv), (B, H, dk, dv), (P, B, H, dk, dv)], 70))
    desc = zeco.make_desc(q, v, g, P, 64, 0.5)
    L_ = zeco.lib()
    calls = [("zeco_gla_local_state", (k, v, g), lambda: (f32(P, B, H, dk, dv), f32(P, B, H, dk))),
             ("zeco_gla_fwd_from_state", (q, k, v, g, S), lambda: (torch.empty_like(v),)),
             ("zeco_gla_bwd_dstate", (q, g, dO), lambda: (f32(P, B, H, dk, dv),)),
             ("zeco_gla_bwd_from_state", (q, k, v, g, dO, S, S_last, dS),
              lambda: (torch.empty_like(q), torch.empty_like(k), torch.empty_like(v), f32(*g.shape)))]
    for c, (name, ins, outs) in enumerate(calls):
        need = L_.zeco_gla_block_workspace(ctypes.byref(desc), c)
        arena = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
        ref = outs()
        _whole(desc, name, ins + ref)
        few = [(arena.data_ptr(), need - 1)]
        if c < 3:   # (the fourth needs one for its checkpoints: null or misaligned is refused)
            few += [(None, 0), (None, need), (arena.data_ptr() + 4, need), (arena.data_ptr(), 0)]
        for ptr, n in few:
            got = outs()
            st = getattr(L_, name + "_ws")(ctypes.byref(desc), *[x.data_ptr() for x in ins + got], ptr, n, zeco._stream())
            torch.cuda.synchronize()
            assert st == zeco.ZECO_OK and all(torch.equal(x, y) for x, y in zip(got, ref)), (name, n)
        got = outs()
        st = getattr(L_, name + "_ws")(ctypes.byref(desc), *[x.data_ptr() for x in ins + got], arena.data_ptr(), need, zeco._stream())
        torch.cuda.synchronize()
        assert st == zeco.ZECO_OK and not all(torch.equal(x, y) for x, y in zip(got, ref)), name   # (that size does cut)
    args = [x.data_ptr() for x in calls[3][1] + calls[3][2]()]
    ck = L_.zeco_gla_bwd_from_state_workspace(ctypes.byref(desc))
    for ptr, n, status in ((None, need, zeco.ZECO_ERR_INVALID_ARG), (arena.data_ptr() + 4, need, zeco.ZECO_ERR_INVALID_ARG),
                           (arena.data_ptr(), ck - 1, zeco.ZECO_ERR_WORKSPACE)):
        assert L_.zeco_gla_bwd_from_state_ws(ctypes.byref(desc), *args, ptr, n, zeco._stream()) == status


def _desc(**kw):
    d = dict(B=1, P=2, H=2, L=4096, d_k=128, d_v=128, C=64, io_dtype=zeco.ZECO_BF16, g_dtype=zeco.ZECO_F32, scale=1.0,
             stride_b=2 * 4096 * 128 * 2, stride_t=256, stride_h=128, vstride_b=2 * 4096 * 128 * 2, vstride_t=256,
             vstride_h=128, g_per_head=0, wide_gates=0)
    d.update(kw)
    return zeco.GlaDesc(*[d[f[0]] for f in zeco.GlaDesc._fields_])


def test_workspace_of_the_blocks():
    L = zeco.lib()

    def ws(call, **kw):
        return L.zeco_gla_block_workspace(ctypes.byref(_desc(**kw)), call)

    state = 4 * 128 * 128
    for call in range(4):
        n = ws(call)
        assert n >= 2 * 2 * 2 * state                            # two pieces a segment at least
        assert n <= (256 * 3 + 64 * 4) * state + (1 << 20)       # states of one round of workgroups; 512 tokens a checkpoint
    # the binding does not even ask beyond these
    for io, C in ((zeco.ZECO_BF16, 64), (zeco.ZECO_F32, 16), (zeco.ZECO_F32, 64)):
        for dk in (64, 128):
            for kw in (dict(P=zeco._BLOCK_STREAMS // 2 + 1), dict(P=1, H=zeco._BLOCK_STREAMS + 1), dict(L=zeco._BLOCK_TOKENS - 1), dict(P=1, H=1, L=64)):
                kw = dict(kw, io_dtype=io, C=C, d_k=dk)
                assert [ws(c, **kw) for c in range(3)] == [0, 0, 0]
                assert ws(3, **kw) == L.zeco_gla_bwd_from_state_workspace(ctypes.byref(_desc(**kw)))
    # nothing to cut: enough streams, short segments, an empty batch; and what is no call or no descriptor
    for kw in (dict(P=65), dict(L=448), dict(B=0)):
        for call in range(3):
            assert ws(call, **kw) == 0
        assert ws(3, **kw) == L.zeco_gla_bwd_from_state_workspace(ctypes.byref(_desc(**kw)))
    assert ws(-1) == 0 and ws(4) == 0 and ws(1, d_k=96) == 0
    # never less than the checkpoints of the whole segments, which is what the call needs to run them whole
    for L_ in (512, 1000, 4096, 1 << 20):
        for H in (1, 2, 16, 32):
            assert ws(3, L=L_, H=H) >= L.zeco_gla_bwd_from_state_workspace(ctypes.byref(_desc(L=L_, H=H)))
