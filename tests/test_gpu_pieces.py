"""The one-call forward and backward cut the whole run of P * L tokens into pieces of whole chunks as even as possible:
lengths where the cut can go wrong (one piece, pieces of one chunk, uneven pieces, a remainder in the last piece,
segments whose ends fall inside pieces), against the oracle's unsegmented recurrence."""
import zlib

import numpy as np
import pytest
import torch

from gpu_util import TOL, host, log_err, rel_err_bh
from oracle import oracle
from paper_2507_01004_amd import synth, zeco

pytestmark = pytest.mark.gpu

#        B, H, P, L, dk, dv, io, gate, C
CASES = [
    (1, 1, 1, 64, 64, 64, "bf16", "f32", 64),        # one chunk, one piece
    (1, 8, 1, 500, 64, 128, "bf16", "f32", 64),      # one piece, ragged: the output pass alone
    (2, 3, 1, 767, 128, 128, "bf16", "bf16", 64),    # few chunks
    (1, 3, 5, 203, 128, 64, "bf16", "f32", 64),      # 15 whole chunks and 55 tokens; segments end inside pieces
    (1, 1, 1, 4159, 64, 128, "bf16", "f32", 64),     # 64 whole chunks and 63 tokens
    (3, 8, 1, 1985, 64, 64, "bf16", "bf16", 64),     # uneven pieces, one token over
    (1, 7, 3, 1100, 128, 128, "bf16", "head", 64),
    (1, 48, 1, 700, 64, 64, "bf16", "head", 64),     # more (batch, head) pairs, few pieces
    (1, 3, 2, 1037, 64, 128, "f32", "f32", 64),
    (1, 2, 3, 333, 128, 64, "f32", "f32", 16),
    (2, 1, 1, 127, 64, 64, "f32", "f32", 32),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d_H%d_P%d_L%d_%dx%d_%s_%s_C%d" % c)
def test_one_call_forward_and_backward_at_the_edges_of_the_cut(case):
    B, H, P, L, dk, dv, io, gate, C = case
    print("case", case, flush=True)
    tol, T, head = TOL[io], P * L, gate == "head"
    seed = zlib.crc32(repr(case).encode()) % 10000
    inp = synth.make_inputs(B, T, H, dk, dv, seed=seed, io=io, g="f32" if head else gate, device="cuda", gate_div=64.0,
                            per_head_gate=head)
    q, k, v, g = (inp[n] for n in "qkvg")
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    dO = torch.randn(v.shape, generator=gen, device="cuda").to(v.dtype)
    S0 = torch.randn(B, H, dk, dv, device="cuda", generator=gen) * 0.3
    dS_T = torch.randn(B, H, dk, dv, device="cuda", generator=gen) * 0.3
    hg = np.repeat(host(g)[..., None], dk, axis=-1) if head else host(g)
    args = (host(q), host(k), host(v), hg)
    for s0 in (None, S0):
        o_r, S_r = oracle.gla_recurrent(*args, 0.5, None if s0 is None else host(s0))
        ref = oracle.gla_recurrent_bwd(*args, host(dO), 0.5, None if s0 is None else host(s0), host(dS_T))
        ref_dg = ref[3].sum(axis=-1) if head else ref[3]
        scheds = (zeco.SCHEDULE_TWO_PHASE, zeco.SCHEDULE_CORRECT) if io == "bf16" else (zeco.SCHEDULE_AUTO,)
        for sched in scheds:
            save = torch.empty(zeco.saved_states_bytes(q, v, g, P, C), dtype=torch.uint8, device="cuda") if io == "bf16" else None
            o, S_last = zeco.gla_fused_fwd(q, k, v, g, P, scale=0.5, S0=s0, C=C, save=save, schedule=sched)
            torch.cuda.synchronize()
            assert rel_err_bh(host(o), o_r, (0, 2)) <= tol and rel_err_bh(host(S_last), S_r, (0, 1)) <= tol
            for saved in {None, save}:
                got = zeco.gla_fused_bwd(q, k, v, g, dO, P, scale=0.5, S0=None if saved is not None else s0, dS_T=dS_T, C=C, saved=saved)
                torch.cuda.synchronize()
                for nm, x, r in zip(("dq", "dk", "dv"), got[:3], ref[:3]):
                    assert rel_err_bh(host(x), r, (0, 2)) <= tol, nm
                assert rel_err_bh(host(got[3]), ref_dg, (0, 2)) <= tol, "dg"
                assert rel_err_bh(host(got[4]), ref[4], (0, 1)) <= tol, "dS0"


VARLEN = [
    # lengths (one over 2112 tokens, so that the call cuts), tokens before the first segment, H, dk, dv, io, gate, C
    ((2113, 64, 700, 65), 0, 2, 128, 128, "bf16", "f32", 64),
    ((100, 3001, 64), 37, 3, 64, 128, "bf16", "head", 64),
    ((64, 64, 2500), 64, 1, 128, 64, "bf16", "bf16", 64),
    ((2200, 129), 5, 2, 64, 64, "f32", "f32", 32),
    ((64,) * 30 + (2176,), 0, 16, 64, 64, "bf16", "f32", 64),     # more segments than pieces
]


@pytest.mark.parametrize("case", VARLEN, ids=lambda c: "%dsegs_%d_H%d_%dx%d_%s_%s" % (len(c[0]), c[1], *c[2:7]))
def test_one_call_over_long_unequal_segments(case):
    """The calls that cut on the device, against the oracle over the tokens the table covers; the others stay as they
    are.  Then the same captured in a graph and replayed with other tables: one with the same lengths in another
    order, one with a segment that is too short, whose rows stay as they are while the segments before it, which it
    cannot touch, come out as without it."""
    lengths, lead, H, dk, dv, io, gate, C = case
    print("case", case, flush=True)
    tol, head, T = TOL[io], gate == "head", lead + sum(lengths) + 11
    seed = zlib.crc32(repr(case).encode()) % 10000
    inp = synth.make_inputs(1, T, H, dk, dv, seed=seed, io=io, g="f32" if head else gate, device="cuda", gate_div=64.0,
                            per_head_gate=head)
    q, k, v, g = (inp[n] for n in "qkvg")
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    dO = torch.randn(v.shape, generator=gen, device="cuda").to(v.dtype)
    S0 = torch.randn(1, H, dk, dv, device="cuda", generator=gen) * 0.3
    dS_T = torch.randn(1, H, dk, dv, device="cuda", generator=gen) * 0.3
    a, e = lead, lead + sum(lengths)
    hg = np.repeat(host(g)[..., None], dk, axis=-1) if head else host(g)
    args = [np.ascontiguousarray(x[:, a:e]) for x in (host(q), host(k), host(v), hg)]
    o_r, S_r = oracle.gla_recurrent(*args, 0.5, host(S0))
    ref = oracle.gla_recurrent_bwd(*args, np.ascontiguousarray(host(dO)[:, a:e]), 0.5, host(S0), host(dS_T))
    ref_dg = ref[3].sum(axis=-1) if head else ref[3]
    mark = 77.0
    seg = torch.tensor([lead] + [lead + int(x) for x in np.cumsum(lengths)], dtype=torch.int64, device="cuda")
    o, S_last = torch.empty_like(v), torch.empty_like(S0)
    grads = (torch.empty_like(q), torch.empty_like(k), torch.empty_like(v), torch.empty(g.shape, device="cuda"), torch.empty_like(S0))
    bound = max(lengths)
    desc = zeco._varlen_desc(q, v, zeco._dtype_code(g), head, seg, bound, 0.5, C)
    L = zeco.lib()
    ws_f, ws_b = (torch.zeros(int(n(zeco.ctypes.byref(desc))), dtype=torch.uint8, device="cuda")
                  for n in (L.zeco_gla_fused_fwd_varlen_workspace, L.zeco_gla_fused_bwd_varlen_workspace))

    def run():
        zeco.gla_fused_fwd_varlen(q, k, v, g, seg, bound, scale=0.5, C=C, S0=S0, out=(o, S_last), workspace=ws_f)
        zeco.gla_fused_bwd_varlen(q, k, v, g, dO, seg, bound, scale=0.5, C=C, S0=S0, dS_T=dS_T, out=grads, workspace=ws_b)

    def check():
        torch.cuda.synchronize()
        assert rel_err_bh(host(o)[:, a:e], o_r, (0, 2)) <= tol and rel_err_bh(host(S_last), S_r, (0, 1)) <= tol
        for nm, x, r in zip(("dq", "dk", "dv", "dg"), grads, ref[:3] + (ref_dg,)):
            assert rel_err_bh(host(x)[:, a:e], r, (0, 2)) <= tol, nm
        assert rel_err_bh(host(grads[4]), ref[4], (0, 1)) <= tol
        for x in (o,) + grads[:4]:
            assert torch.all(x[:, :a] == mark) and torch.all(x[:, e:] == mark)

    for x in (o,) + grads[:4]:
        x.fill_(mark)
    run()
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for order in (lengths, lengths[::-1]):
        seg.copy_(torch.tensor([lead] + [lead + int(x) for x in np.cumsum(order)], dtype=torch.int64))
        for x in (o,) + grads[:4]:
            x.fill_(mark)
        graph.replay()
        check()
    good = o.clone()
    seg[-2] = e - 40                      # the last segment breaks the rules, and perhaps the one before it (too long)
    o.fill_(mark)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.all(o[:, e - 40:] == mark)
    n = int(seg[-3]) if len(lengths) > 2 else a
    assert (o[:, a:n].float() - good[:, a:n].float()).abs().max().item() <= tol * good.float().abs().max().item() if n > a else True


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("C", [16, 32, 64])
def test_fp32_passes_at_chunk_edges(C, dk, dv):
    """The fp32 kernels' thread mappings (16-byte loads, token groups per wave) for every tile shape: three calls and the
    two fp32 directions over segments one token short of, at and one token past a multiple of the chunk."""
    B, H, P = 1, 2, 2
    for L in (64 + C - 1, 128, 64 + C + 1):
        print("case", C, dk, dv, L, flush=True)
        inp = synth.make_inputs(B, P * L, H, dk, dv, seed=500 + L, io="f32", g="f32", device="cuda", gate_div=32.0)
        q, k, v, g = (inp[n] for n in "qkvg")
        gen = torch.Generator(device="cuda").manual_seed(L)
        dO = torch.randn(v.shape, generator=gen, device="cuda")
        S0 = torch.randn(B, H, dk, dv, device="cuda", generator=gen) * 0.3
        args = [host(x) for x in (q, k, v, g)]
        o_r, S_r = oracle.gla_recurrent(*args, 0.5, host(S0))
        o, S_last, _ = zeco.segmented_fwd(q, k, v, g, P, scale=0.5, S0=S0, C=C)
        ref = oracle.gla_recurrent_bwd(*args, host(dO), 0.5, host(S0))
        got = zeco.gla_fused_bwd(q, k, v, g, dO, P, scale=0.5, S0=S0, C=C)
        torch.cuda.synchronize()
        assert rel_err_bh(host(o), o_r, (0, 2)) <= TOL["f32"] and rel_err_bh(host(S_last), S_r, (0, 1)) <= TOL["f32"]
        for nm, x, r in zip(("dq", "dk", "dv", "dg"), got, ref):
            assert rel_err_bh(host(x), r, (0, 2)) <= TOL["f32"], nm


@pytest.mark.parametrize("case", [(1, 3, 2, 1700, 128, 128, "bf16", "f32"), (2, 1, 1, 2111, 64, 128, "bf16", "bf16"), (1, 5, 3, 1089, 128, 64, "bf16", "head"),
                                  (1, 21, 1, 831, 64, 64, "bf16", "f32"), (1, 1, 7, 512, 128, 128, "bf16", "f32"), (1, 2, 3, 1111, 64, 128, "f32", "f32"),
                                  (2, 1, 1, 640, 128, 64, "f32", "f32")], ids=lambda c: "B%d_H%d_P%d_L%d_%dx%d_%s_%s" % c)
def test_local_pass_of_few_streams_at_odd_lengths(case):
    """The local pass cuts segments of few streams into sub-segments that need not be equal: every output of it, and the
    three calls together, against the oracle."""
    B, H, P, L, dk, dv, io, gate = case
    print("case", case, flush=True)
    head, tol = gate == "head", TOL[io]
    inp = synth.make_inputs(B, P * L, H, dk, dv, seed=L, io=io, g="f32" if head else gate, device="cuda", gate_div=64.0,
                            per_head_gate=head)
    q, k, v, g = (inp[n] for n in "qkvg")
    S0 = torch.randn(B, H, dk, dv, device="cuda", generator=torch.Generator(device="cuda").manual_seed(L)) * 0.3
    hg = np.repeat(host(g)[..., None], dk, axis=-1) if head else host(g)
    args = (host(q), host(k), host(v), hg)
    o_l, S_l, Gc_l, Gt_l = oracle.gla_local(*args, P, 0.5)
    o, S_loc, G_cum, G_tot = zeco.gla_local_fwd(q, k, v, g, P, scale=0.5)
    torch.cuda.synchronize()
    assert rel_err_bh(host(o), o_l, (0, 2)) <= tol and rel_err_bh(host(S_loc), S_l, (1, 2)) <= tol
    assert log_err(host(G_cum), Gc_l[..., 0] if head else Gc_l) <= 1e-5
    assert log_err(host(G_tot), Gt_l[..., 0] if head else Gt_l) <= 1e-5
    o, S_last, _ = zeco.segmented_fwd(q, k, v, g, P, scale=0.5, S0=S0)
    o_r, S_r = oracle.gla_recurrent(*args, 0.5, host(S0))
    torch.cuda.synchronize()
    assert rel_err_bh(host(o), o_r, (0, 2)) <= tol and rel_err_bh(host(S_last), S_r, (0, 1)) <= tol
    if io == "f32":   # a smaller workspace: the segments whole
        whole = zeco.gla_local_fwd(q, k, v, g, P, scale=0.5, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert rel_err_bh(host(whole[0]), o_l, (0, 2)) <= tol and log_err(host(whole[2]), Gc_l) <= 1e-5


@pytest.mark.parametrize("case", [(1, 2, 1, 20011, 64, 64, "bf16", "f32"), (1, 3, 2, 4097, 128, 128, "bf16", "bf16"), (1, 5, 1, 8191, 64, 128, "bf16", "head"),
                                  (1, 2, 1, 20011, 64, 64, "f32", "f32"), (2, 1, 2, 4096, 128, 64, "f32", "f32")], ids=lambda c: "B%d_H%d_P%d_L%d_%dx%d_%s_%s" % c)
def test_log_decays_of_a_cut_segment_are_those_of_one_chain(case):
    """A segment's cumulative log decay keeps the bits fp32 cannot hold from chunk to chunk, so that every G_cum is one sum
    rounded to fp32; cut into sub-segments it is the same sum.  The cut ends where the whole segment's chunks end, so the
    two differ only where the extended sums fall on different sides of a rounding boundary, and by one unit: in fp32
    calls the extended sums hold 48 bits (about one value in 2^20; allowed one in 1000).  In bf16 calls a chunk's total,
    below 8, joins the pair rounded to its own last place, by up to 2^-22: a random sum of 2^-23 sqrt(N) after N chunks,
    where fp32 values are 2^-17 apart at sums of a hundred (16 chunks, 1 : 16) and 2^-13 at sums of two thousand (313
    chunks, 1 : 60): allowed one value in 60.  A prefix rounded to fp32 moves by a quarter of a unit on average."""
    B, H, P, L, dk, dv, io, gate = case
    print("case", case, flush=True)
    inp = synth.make_inputs(B, P * L, H, dk, dv, seed=L, io=io, g="f32" if gate == "head" else gate, device="cuda", gate_div=8.0,
                            per_head_gate=gate == "head")
    q, k, v, g = (inp[n] for n in "qkvg")
    assert zeco.local_fwd_workspace_bytes(q, v, g, P) > 0          # the call cuts
    cut = zeco.gla_local_fwd(q, k, v, g, P)
    whole = zeco.gla_local_fwd(q, k, v, g, P, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    for nm, a, b in (("G_cum", cut[2], whole[2]), ("G_tot", cut[3], whole[3])):
        other = (a != b).double().mean().item()
        print(nm, "differ", other, flush=True)
        assert other <= max(1e-3 if io == "f32" else 1 / 60, 1.0 / a.numel()), nm
        assert ((a - b).abs() <= b.abs() * 2.0 ** -22).all(), nm


@pytest.mark.parametrize("B,H,P,L", [(1, 8, 64, 2048), (1, 16, 64, 1000), (1, 1, 1, 70001), (2, 8, 1, 100001)])
def test_the_cut_brings_no_call_to_the_correction(B, H, P, L):
    """AUTO corrects only where the caller's own segments are long: short segments, and a single run whose odd length does
    not halve, stay with the two phases (o rounded once, a time that does not depend on the decays), however long the
    pieces of the library's cut are."""
    print("case", B, H, P, L, flush=True)
    inp = synth.make_inputs(B, P * L, H, 64, 64, seed=L, io="bf16", g="bf16", device="cuda", gate_div=512.0)
    q, k, v, g = (inp[n] for n in "qkvg")
    auto, _ = zeco.gla_fused_fwd(q, k, v, g, P)
    two, _ = zeco.gla_fused_fwd(q, k, v, g, P, schedule=zeco.SCHEDULE_TWO_PHASE)
    torch.cuda.synchronize()
    assert torch.equal(auto, two)


@pytest.mark.parametrize("io,L", [("f32", 1024), ("f32", 1111), ("bf16", 1111), ("bf16", 576)])
def test_local_pass_runs_whole_with_a_workspace_it_cannot_use(io, L):
    """Where the local pass can do without a workspace it takes whatever it is given: nothing, too few bytes, or enough of
    them at an address it cannot use - and then runs every segment as one chain."""
    print("case", io, L, flush=True)
    inp = synth.make_inputs(1, 2 * L, 2, 64, 64, seed=L, io=io, g="f32", device="cuda", gate_div=64.0)
    q, k, v, g = (inp[n] for n in "qkvg")
    n = zeco.local_fwd_workspace_bytes(q, v, g, 2)
    assert n > 0
    whole = zeco.gla_local_fwd(q, k, v, g, 2, workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
    for ws in (torch.empty(n - 1, dtype=torch.uint8, device="cuda"), torch.empty(n + 8, dtype=torch.uint8, device="cuda")[8:]):
        got = zeco.gla_local_fwd(q, k, v, g, 2, workspace=ws)
        torch.cuda.synchronize()
        for a, b in zip(got, whole):
            assert torch.equal(a, b)


def checkpoints_per_piece(q, v, g, P, C):
    """(pieces, checkpoints of the forward state a piece has) of a one-call backward, from what its workspace holds:
    four states a piece, one more and the pieces' log decays, and a state per checkpoint, one every eight chunks of 64
    tokens (the count that gives that size)."""
    B, T, H, dk = q.shape
    dv, chunks, ws = v.shape[-1], T // 64, zeco.fused_bwd_workspace_bytes(q, v, g, P, C) // 4
    found = []
    for n in range(1, chunks + 1):
        longest = 64 * (chunks // n + 1) if chunks % n else 64 * (chunks // n) + T % 64
        ck = ((longest + 63) // 64 - 1) // 8
        if B * H * (n * (4 * dk * dv + dk + ck * dk * dv) + dk * dv) == ws:
            found.append((n, ck))
    assert len(found) == 1, found
    return found[0]


CHECKPOINTED = [(1, 16, 1, 9507, 64, 64, "bf16", "f32", 64), (1, 16, 3, 3169, 64, 128, "bf16", "head", 64), (1, 16, 1, 9507, 64, 64, "f32", "f32", 64),
                (1, 64, 1, 4901, 64, 64, "f32", "f32", 32), (1, 64, 1, 4901, 64, 64, "f32", "f32", 16)]


@pytest.mark.parametrize("case", CHECKPOINTED, ids=lambda c: "B%d_H%d_P%d_L%d_%dx%d_%s_%s_C%d" % c)
def test_one_call_backward_over_pieces_with_checkpoints(case):
    """Uneven pieces of nine chunks or more, so that dG is re-anchored inside them from the forward states the dQ pass
    left (and the saved states, with bf16, start the backward), against the oracle."""
    B, H, P, L, dk, dv, io, gate, C = case
    print("case", case, flush=True)
    tol, head = TOL[io], gate == "head"
    seed = zlib.crc32(repr(case).encode()) % 10000
    inp = synth.make_inputs(B, P * L, H, dk, dv, seed=seed, io=io, g="f32", device="cuda", gate_div=64.0, per_head_gate=head)
    q, k, v, g = (inp[n] for n in "qkvg")
    n, ck = checkpoints_per_piece(q, v, g, P, C)
    assert ck >= 1 and (P * L // 64) % n
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    dO = torch.randn(v.shape, generator=gen, device="cuda").to(v.dtype)
    S0 = torch.randn(B, H, dk, dv, device="cuda", generator=gen) * 0.3
    dS_T = torch.randn(B, H, dk, dv, device="cuda", generator=gen) * 0.3
    hg = np.repeat(host(g)[..., None], dk, axis=-1) if head else host(g)
    ref = oracle.gla_recurrent_bwd(host(q), host(k), host(v), hg, host(dO), 0.5, host(S0), host(dS_T))
    ref_dg = ref[3].sum(axis=-1) if head else ref[3]
    save = None
    if io == "bf16":
        save = torch.empty(zeco.saved_states_bytes(q, v, g, P, C), dtype=torch.uint8, device="cuda")
        zeco.gla_fused_fwd(q, k, v, g, P, scale=0.5, S0=S0, C=C, save=save)
    for saved in {None, save}:
        got = zeco.gla_fused_bwd(q, k, v, g, dO, P, scale=0.5, S0=None if saved is not None else S0, dS_T=dS_T, C=C, saved=saved)
        torch.cuda.synchronize()
        for nm, x, r in zip(("dq", "dk", "dv", "dg"), got[:4], ref[:3] + (ref_dg,)):
            assert rel_err_bh(host(x), r, (0, 2)) <= tol, nm
        assert rel_err_bh(host(got[4]), ref[4], (0, 1)) <= tol, "dS0"


@pytest.mark.parametrize("lengths,lead,H,dk,dv,io,gate,C", [((3001, 64, 2113, 700, 3629), 37, 16, 64, 64, "bf16", "f32", 64),
                                                           ((2500, 64, 2337), 5, 64, 64, 64, "f32", "f32", 16)])
def test_one_call_backward_over_a_table_with_checkpoints(lengths, lead, H, dk, dv, io, gate, C):
    """The same over a table of unequal segments: the checkpoints a piece has, and their places, come from the device."""
    print("case", lengths, lead, H, dk, dv, io, gate, C, flush=True)
    tol, T = TOL[io], lead + sum(lengths) + 11
    inp = synth.make_inputs(1, T, H, dk, dv, seed=len(lengths), io=io, g="f32", device="cuda", gate_div=64.0)
    q, k, v, g = (inp[n] for n in "qkvg")
    a, e = lead, lead + sum(lengths)
    run = [x[:, a:e] for x in (q, v, g)]
    n, ck = checkpoints_per_piece(*run, 1, C)     # the run's pieces: the table's calls cut it by the same estimate
    assert ck >= 1 and (sum(lengths) // 64) % n
    gen = torch.Generator(device="cuda").manual_seed(7)
    dO = torch.randn(v.shape, generator=gen, device="cuda").to(v.dtype)
    S0 = torch.randn(1, H, dk, dv, device="cuda", generator=gen) * 0.3
    seg = torch.tensor([lead] + [lead + int(x) for x in np.cumsum(lengths)], dtype=torch.int64, device="cuda")
    ref = oracle.gla_recurrent_bwd(*(np.ascontiguousarray(host(x)[:, a:e]) for x in (q, k, v, g, dO)), 0.5, host(S0))
    got = zeco.gla_fused_bwd_varlen(q, k, v, g, dO, seg, max(lengths), scale=0.5, C=C, S0=S0)
    torch.cuda.synchronize()
    for nm, x, r in zip(("dq", "dk", "dv", "dg"), got, ref):
        assert rel_err_bh(host(x)[:, a:e], r, (0, 2)) <= tol, nm
    assert rel_err_bh(host(got[4]), ref[4], (0, 1)) <= tol
