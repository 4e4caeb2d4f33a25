"""The kernels that take whole chunks, forwards and backwards.  The single-launch forward kernels (a span's chunks on chip from the first
load to the last store, states handed on through flags) at their edges: head sizes around the 16-channel units, the tail and the
16-column tiles, groups of 4 and of 8 chunks, filled or not, ragged last chunks and spans, grids whose columns are shorter than a tile,
both memory orders, an initial state, slow gates (every earlier span is looked at), sums over scan orders, gate prologue and epilogue;
a wait that runs out, and replays of a graph.

Tolerance: as for the other kernels with split operands, 2e-4 of the RMS (an operand pair carries 16 bits, a product is off by at
most 4 * 2^-17 of itself, and an output's largest value is about six times its RMS); a bf16 store adds at most half a unit of its
eighth bit, 2^-8 of the largest value.  The epilogue divides rows by their spread: 2e-3."""
import numpy as np
import pytest
import torch

import paper_2405_18428_amd as gla
from paper_2405_18428_amd import inputs as gi

pytestmark = pytest.mark.gpu
TOL = 2e-4
POLLS = 1 << 15


@pytest.fixture(autouse=True)
def defaults():
    yield
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    gla.gla_set_option(gla.OPT_LOOK_BACK_POLLS, POLLS)


def upload(d, *names):
    f = lambda n: torch.from_numpy(d[n + "_bits"].view(np.int16)).cuda().view(torch.bfloat16)
    return [torch.from_numpy(d[n]).cuda() if n == "log_alpha" else f(n) for n in names]


def near(got, want, bf16=False, tol=TOL):
    got, rms, top = got.float().cpu().numpy(), np.sqrt(np.mean(want ** 2)), np.abs(want).max()
    assert np.abs(got - want).max() / rms <= tol * max(1.0, top / rms / 6) + (2.0 ** -8 * top / rms if bf16 else 0.0)


# (sequences as B x H, grid): one span; spans of two chunks with a ragged last one; of 4 (small heads 3); of 4 with a last span of one
# chunk; full ones; spans of 5 in groups that could hold 8, with a last one of two chunks and with none; two rounds of groups;
# one span of 6 chunks; many sequences of four (small heads)
PLANS = [(2, 2, 16, 16), (4, 16, 50, 7), (2, 16, 3, 365), (1, 6, 97, 64), (8, 16, 5, 91), (4, 16, 64, 17), (8, 16, 4, 151), (6, 16, 25, 43),
         (2, 16, 100, 65), (10, 16, 5, 72), (16, 16, 8, 30)]


@pytest.mark.parametrize("dk,dv,B,H,gh,gw", [(*h, *c) for h in ((36, 72), (32, 64)) for c in PLANS] +
                         [(*h, *c) for h in ((20, 40), (36, 40), (28, 72)) for c in PLANS[:5]])
def test_plans_and_heads(dk, dv, B, H, gh, gw):
    from oracle import gla_oracle
    d = gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=dk + dv + gh, z_mean=3.0 if gw % 2 else 0.0)
    s0 = np.random.default_rng(5).standard_normal((B, H, dk, dv)).astype(np.float32)
    for scan, layout, out_dtype in ((1, 0, torch.float32), (2, 1, torch.bfloat16)):
        ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, scan, initial_state=s0)
        t = upload(d, "q", "k", "v", "log_alpha")
        if layout == 1:
            t = [x.transpose(1, 2).contiguous() for x in t]
        out, fin = gla.gla_fwd_layout(*t, gh, gw, scan, layout=layout, initial_state=torch.from_numpy(s0).cuda(), out_dtype=out_dtype)
        near(out if layout == 0 else out.transpose(1, 2), ref, out_dtype == torch.bfloat16)
        near(fin, ref_fin)


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("B,H,gh,gw,scans", [(4, 16, 50, 7, (0, 3)), (2, 16, 64, 64, (1, 2))])
def test_sums_and_their_states(B, H, gh, gw, scans, dk, dv):
    """Sums over scan orders; the last order's span states serve the backward call."""
    from oracle import gla_oracle
    d = gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=6)
    t = upload(d, "q", "k", "v", "log_alpha")
    ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    out = gla.gla_fwd_multi(*t, gh, gw, scan_dirs=scans, workspace=ws)
    near(out, sum(gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, s)[0] for s in scans))
    w = torch.randn(B, H, gh * gw, dv, device="cuda").bfloat16()
    for got, own in zip(gla.gla_bwd(*t, w, gh, gw, scans[-1], fwd_workspace=ws)[:3], gla.gla_bwd(*t, w, gh, gw, scans[-1])[:3]):
        near(got, own.cpu().numpy(), tol=2 * TOL)       # (two sums over other spans)


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64), (20, 40)])
@pytest.mark.parametrize("B,H,gh,gw", [(2, 3, 16, 15), (4, 16, 40, 13), (8, 16, 23, 37), (16, 16, 8, 61), (2, 3, 11, 16), (2, 6, 13, 41), (12, 16, 35, 22),
                                       (24, 16, 15, 34)])
def test_gate_prologue_and_epilogue(B, H, gh, gw, dk, dv):
    from oracle import gla_oracle_fused as fo
    d = gi.make_fused_inputs(B, H, gh * gw, dk, dv, "bf16", seed=7)
    q, k, v, z, r = upload(d, "q", "k", "v", "z", "r")
    lnw, lnb = (torch.from_numpy(d[n]).cuda() for n in ("ln_w", "ln_b"))
    for scan, out_dtype in ((0, torch.float32), (3, torch.bfloat16)):
        ref, ref_fin = fo.gla_fused(d["q"], d["k"], d["v"], d["z"], 16.0, None, None, None, 1e-5, gh, gw, scan)
        gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_MFMA)
        out, fin = gla.gla_fwd_fused(q, k, v, z, 16.0, gh, gw, scan, out_dtype=out_dtype)
        near(out, ref, out_dtype == torch.bfloat16)
        near(fin, ref_fin)
        ref, _ = fo.gla_fused(d["q"], d["k"], d["v"], d["z"], 16.0, d["r"], d["ln_w"], d["ln_b"], 1e-5, gh, gw, scan)
        out, fin = gla.gla_fwd_fused(q, k, v, z, 16.0, gh, gw, scan, r_pre=r, ln_weight=lnw, ln_bias=lnb, ln_eps=1e-5, out_dtype=out_dtype)
        near(out, ref, out_dtype == torch.bfloat16, tol=2e-3)
        near(fin, ref_fin)


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64), (20, 40), (36, 40), (28, 72)])
@pytest.mark.parametrize("B,H,gh,gw", [(2, 3, 16, 15), (4, 8, 5, 117), (2, 16, 64, 11), (8, 16, 9, 65)])
def test_two_sided_gate(dk, dv, B, H, gh, gw):
    """One span, spans of four chunks with a last one of one token or one chunk, two rounds of groups; both memory orders, an
    initial state, no polls in one of them."""
    from oracle import gla_oracle_gates as go
    d = gi.make_gate_inputs(B, H, gh * gw, dk, dv, "bf16", seed=dk + gh)
    s0 = np.random.default_rng(5).standard_normal((B, H, dk, dv)).astype(np.float32)
    for scan, layout, out_dtype, polls in ((1, 0, torch.float32, POLLS), (2, 1, torch.bfloat16, POLLS), (0, 0, torch.float32, 0)):
        if polls == 0 and gh * gw * B * H > 25000:
            continue        # (what the wait leaves to be formed from the inputs takes its time)
        gla.gla_set_option(gla.OPT_LOOK_BACK_POLLS, polls)
        ref, ref_fin = go.gla_fwd_gates(d["q"], d["k"], d["v"], d["log_alpha"], d["log_beta"], gh, gw, scan, initial_state=s0)
        t = upload(d, "q", "k", "v", "log_alpha") + [torch.from_numpy(d["log_beta"]).cuda()]
        if layout == 1:
            t = [x.transpose(1, 2).contiguous() for x in t]
        out, fin = gla.gla_fwd_gates(*t, gh, gw, scan, layout=layout, initial_state=torch.from_numpy(s0).cuda(), out_dtype=out_dtype)
        near(out if layout == 0 else out.transpose(1, 2), ref, out_dtype == torch.bfloat16)
        near(fin, ref_fin)


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("scan", [0, 3])
def test_a_wait_that_runs_out(scan, fused):
    """No polls at all: what a span does not find at once it forms from the inputs."""
    from oracle import gla_oracle
    B, H, gh, gw, dk, dv = 1, 7, 20, 254, 36, 72
    d = gi.make_fused_inputs(B, H, gh * gw, dk, dv, "bf16", seed=8)
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_MFMA)
    gla.gla_set_option(gla.OPT_LOOK_BACK_POLLS, 0)
    q, k, v, z = upload(d, "q", "k", "v", "z")
    la = torch.nn.functional.logsigmoid(z.float()) / 16
    ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], la.cpu().numpy(), gh, gw, scan)
    for _ in range(2):
        out, fin = gla.gla_fwd_fused(q, k, v, z, 16.0, gh, gw, scan) if fused else gla.gla_fwd_ex(q, k, v, la, gh, gw, scan)
        near(out, ref)
        near(fin, ref_fin)


@pytest.mark.parametrize("dk,dv,B,H,gh,gw", [(36, 72, 4, 25, 24, 24), (32, 64, 4, 25, 24, 24), (20, 40, 4, 25, 9, 61), (32, 64, 2, 8, 20, 64)])
def test_a_wait_that_runs_out_in_other_kernels(dk, dv, B, H, gh, gw):
    """The same in groups of eight (100 sequences of nine chunks, two spans) and, of small heads, of four: an initial state in [B,T,H,d], sums
    over scan orders, and the epilogue, whose rows are on their way to LDS meanwhile.  Waits that end well give the same."""
    from oracle import gla_oracle, gla_oracle_fused as fo
    d = gi.make_fused_inputs(B, H, gh * gw, dk, dv, "bf16", seed=dk + gw)
    s0 = np.random.default_rng(5).standard_normal((B, H, dk, dv)).astype(np.float32)
    q, k, v, z, r = upload(d, "q", "k", "v", "z", "r")
    lnw, lnb = (torch.from_numpy(d[n]).cuda() for n in ("ln_w", "ln_b"))
    la = torch.nn.functional.logsigmoid(z.float()) / 16
    log_alpha = la.cpu().numpy()
    order = lambda s, **more: gla_oracle.gla_fwd(d["q"], d["k"], d["v"], log_alpha, gh, gw, s, **more)
    want, want_fin = order(3, initial_state=s0)
    total = order(0)[0] + order(2)[0]
    mixed, mixed_fin = fo.gla_fused(d["q"], d["k"], d["v"], d["z"], 16.0, d["r"], d["ln_w"], d["ln_b"], 1e-5, gh, gw, 1)
    for polls in (0, POLLS):
        gla.gla_set_option(gla.OPT_LOOK_BACK_POLLS, polls)
        t = [x.transpose(1, 2).contiguous() for x in (q, k, v, la)]
        out, fin = gla.gla_fwd_layout(*t, gh, gw, 3, layout=1, initial_state=torch.from_numpy(s0).cuda())
        near(out.transpose(1, 2), want)
        near(fin, want_fin)
        near(gla.gla_fwd_multi(q, k, v, la, gh, gw, scan_dirs=[0, 2]), total)
        out, fin = gla.gla_fwd_fused(q, k, v, z, 16.0, gh, gw, 1, r_pre=r, ln_weight=lnw, ln_bias=lnb, ln_eps=1e-5)
        near(out, mixed, tol=2e-3)
        near(fin, mixed_fin)


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("step", [0, 20, 31, 32, 63])
@pytest.mark.parametrize("B,H,chunks", [(1, 16, 4), (1, 16, 40)])
def test_gate_of_exactly_zero(dk, dv, B, H, chunks, step):
    """log_alpha = -inf (a pre-activation as low; log_beta = -inf) on some channels at one step: the limits of the operands do not cover it, but
    nothing is lost to NaN, and what does not hang on that chunk is right: outputs and dq from seven chunks on, whose earlier steps have decayed to
    less than TOL, dk and dv of the chunks behind it."""
    from oracle import gla_oracle, gla_oracle_gates as go
    gh, gw = chunks, 64
    at, behind = 64 * (1 if chunks == 4 else 2) + step, 64 * (2 if chunks == 4 else 3)
    d = gi.make_gate_inputs(B, H, gh * gw, dk, dv, "bf16", seed=7)
    open_beta = d["log_beta"].copy()
    d["log_alpha"][:, :, at, [0, 5, 17, 31]] = -np.inf
    d["log_beta"][:, :, at, [1, 16, 39, 63]] = -np.inf
    q, k, v, la = upload(d, "q", "k", "v", "log_alpha")
    z = torch.randn(B, H, gh * gw, dk, device="cuda").bfloat16()
    z[:, :, at, [0, 5, 17, 31]] = -3e38
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, gh * gw, dv)).astype(np.float32)).bfloat16()
    finite = lambda *t: all(bool(torch.isfinite(x).all()) for x in t)
    ws = torch.empty(gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16), dtype=torch.uint8, device="cuda")
    out, fin = gla.gla_fwd_ex(q, k, v, la, gh, gw, 0, workspace=ws)
    assert finite(out, fin)
    assert finite(*gla.gla_fwd_fused(q, k, v, z, 16.0, gh, gw, 0, r_pre=v, ln_eps=1e-5))
    for keep in (None, ws):
        grads = gla.gla_bwd(q, k, v, la, w.cuda(), gh, gw, 0, fwd_workspace=keep)
        assert finite(*grads)
        want = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, 0)
        for g, r in zip(grads[1:3], want[1:3]):
            near(g[:, :, behind:], r[:, :, behind:])
        if chunks > 9:
            near(grads[0][:, :, 9 * 64:], want[0][:, :, 9 * 64:])
    alpha_only = torch.from_numpy(open_beta).cuda()
    open_alpha = np.where(np.isinf(d["log_alpha"]), np.float32(-0.1), d["log_alpha"])
    for a, b, na, nb in ((la, alpha_only, d["log_alpha"], open_beta),
                         (torch.from_numpy(open_alpha).cuda(), torch.from_numpy(d["log_beta"]).cuda(), open_alpha, d["log_beta"])):
        got, got_fin = gla.gla_fwd_gates(q, k, v, a, b, gh, gw, 0)
        assert finite(got, got_fin)
        if chunks > 9:
            ref, ref_fin = go.gla_fwd_gates(d["q"], d["k"], d["v"], na, nb, gh, gw, 0)
            near(got[:, :, 9 * 64:], ref[:, :, 9 * 64:])
            near(got_fin, ref_fin)
    if chunks > 9:
        ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, 0)
        near(out[:, :, 9 * 64:], ref[:, :, 9 * 64:])
        near(fin, ref_fin)


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("B,H,chunks", [(1, 8, 80), (2, 8, 80)])
def test_chain_behind_zeros(dk, dv, B, H, chunks):
    """No keys in the last 60 chunks: what is left of the first ones has decayed far below the 2^-40 at which a chain of span states stops, but it
    is all there is (groups of four and of eight; the gate on both sides).  Backwards the same: no gradient from chunk 4 to 63, so that dv and dk
    of these chunks come from the last ones, and dq of the last from the first."""
    from oracle import gla_oracle, gla_oracle_gates as go
    gh, gw = chunks, 64
    d = gi.make_gate_inputs(B, H, gh * gw, dk, dv, "bf16", seed=21, z_mean=1.5)
    d["k"][:, :, 20 * 64:] = 0.0
    d["k_bits"] = gi.round_to_bf16_bits(d["k"])
    w = np.random.default_rng(9).standard_normal((B, H, gh * gw, dv)).astype(np.float32)
    w[:, :, 4 * 64:64 * 64] = 0.0
    w = torch.from_numpy(w).bfloat16()
    q, k, v, la = upload(d, "q", "k", "v", "log_alpha")
    lb = torch.from_numpy(d["log_beta"]).cuda()
    one, both = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, 0), go.gla_fwd_gates(
        d["q"], d["k"], d["v"], d["log_alpha"], d["log_beta"] / 16, gh, gw, 0)
    assert 0.0 < np.abs(one[1]).max() < 2.0 ** -50 and 0.0 < np.abs(both[1]).max() < 2.0 ** -50
    out, fin = gla.gla_fwd_ex(q, k, v, la, gh, gw, 0)
    last = slice((chunks - 1) * 64, None)
    near(fin, one[1])
    near(out[:, :, last], one[0][:, :, last])
    out, fin = gla.gla_fwd_gates(q, k, v, la, lb / 16, gh, gw, 0)
    near(fin, both[1])
    near(out[:, :, last], both[0][:, :, last])
    want = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, 0)
    got = gla.gla_bwd(q, k, v, la, w.cuda(), gh, gw, 0)
    near(got[0][:, :, last], want[0][:, :, last])
    for g, r in zip(got[1:3], want[1:3]):
        assert 0.0 < np.abs(r[:, :, 8 * 64:9 * 64]).max() < 2.0 ** -50
        near(g[:, :, 8 * 64:9 * 64], r[:, :, 8 * 64:9 * 64])


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("two_sided,bh,chunks", [(False, 36, 112), (True, 50, 32), (False, 12, 288), (True, 40, 64), (True, 12, 128)])
def test_several_rounds(two_sided, bh, chunks, dk, dv):
    """Groups in several rounds, of spans in order (work-groups a multiple of eight, sequences not), in ranges of whole sequences, and in ranges that
    sequences straddle, with slow gates: as the two-pass kernels have it (which GLA_CARRY_KERNEL asks for)."""
    g = torch.Generator(device="cuda").manual_seed(bh)
    T = 64 * chunks
    q, k, v = (torch.randn(1, bh, T, d, generator=g, device="cuda").bfloat16() for d in (dk, dk, dv))
    gate = lambda d: torch.nn.functional.logsigmoid(torch.randn(1, bh, T, d, generator=g, device="cuda") + 4.0) / 16
    more = (gate(dk), gate(dv)) if two_sided else (gate(dk),)
    call = gla.gla_fwd_gates if two_sided else gla.gla_fwd_ex
    try:
        gla.gla_set_option(gla.OPT_CARRY, gla.CARRY_KERNEL)
        gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_MFMA)
        want = [x.cpu().numpy() for x in call(q, k, v, *more, chunks, 64, 2)]
    finally:
        gla.gla_set_option(gla.OPT_CARRY, gla.CARRY_AUTO)
        gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    for got, ref in zip(call(q, k, v, *more, chunks, 64, 2), want):
        near(got, ref, tol=2 * TOL)


def test_two_streams():
    """Calls that wait inside a launch, on two streams at once, each with a workspace of its own: every result as it is alone.  Groups of eight that fill
    the chip beside groups of four, slow gates, so that every group waits; a poll that runs out changes the last bits only."""
    g = torch.Generator(device="cuda").manual_seed(3)
    calls = []
    for bh, chunks, dk, dv in ((16, 100, 36, 72), (6, 120, 32, 64), (16, 256, 36, 72)):
        T = 64 * chunks
        t = [torch.randn(1, bh, T, d, generator=g, device="cuda").bfloat16() for d in (dk, dk, dv)]
        t.append(torch.nn.functional.logsigmoid(torch.randn(1, bh, T, dk, generator=g, device="cuda") + 4.0) / 16)
        ws = torch.empty(gla.gla_fwd_workspace_bytes(1, bh, T, dk, dv, gla.DT_BF16), dtype=torch.uint8, device="cuda")
        calls.append((t, chunks, ws, gla.gla_fwd_ex(*t, chunks, 64, 0, workspace=ws)))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for pair in ((0, 1), (2, 0), (1, 2)):
        torch.cuda.synchronize()
        kept = []
        for _ in range(8):
            for c, stream in zip(pair, streams):
                t, chunks, ws, _want = calls[c]
                with torch.cuda.stream(stream):
                    kept.append((c, gla.gla_fwd_ex(*t, chunks, 64, 0, workspace=ws)))
        torch.cuda.synchronize()
        for c, got in kept:
            for x, ref in zip(got, calls[c][3]):
                assert float((x - ref).abs().max() / ref.square().mean().sqrt()) <= TOL


# (one span of three and of four chunks, ragged; several spans, with a last one of one token and with one of four chunks; two rounds
# of one-span groups; short columns)
BACK = [(2, 3, 14, 13), (2, 3, 3, 84), (1, 6, 16, 16), (18, 16, 5, 37), (8, 16, 11, 35), (2, 16, 9, 57), (4, 16, 64, 15), (16, 16, 32, 7)]


# (129 to 256 sequences of 6, 7 and 8 chunks: one span each in the forward call, several in the walks that follow it)
ONE_SPAN = [(10, 16, 5, 72), (12, 16, 7, 61), (16, 16, 8, 61)]


@pytest.mark.parametrize("dk,dv,B,H,gh,gw", [(*h, *c) for h in ((36, 72), (32, 64)) for c in BACK + ONE_SPAN] +
                         [(*h, *c) for h in ((20, 40), (36, 40), (28, 72)) for c in BACK[:5]])
def test_gradients(dk, dv, B, H, gh, gw):
    """All four gradients, both memory orders, with and without the forward call's workspace; slow gates in every other case.  The gate
    gradient sums up to 64 terms q dq - k dk and two states: 64 TOL of their size, whatever cancels."""
    from oracle import gla_oracle
    d = gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=dk + dv + gh, z_mean=3.0 if gw % 2 else 0.0)
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, gh * gw, dv)).astype(np.float32)).bfloat16()
    for scan, layout in ((2, 0), (1, 1)):
        want = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, scan)
        size = max(np.sqrt(np.mean((d["q"].astype(np.float64) * want[0]) ** 2)), np.sqrt(np.mean(want[3] ** 2)))
        t = upload(d, "q", "k", "v", "log_alpha") + [w.cuda()]
        if layout == 1:
            t = [x.transpose(1, 2).contiguous() for x in t]
        ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
        gla.gla_fwd_layout(*t[:4], gh, gw, scan, layout=layout, workspace=ws)
        for keep in (None, ws):
            room = torch.full((gla.gla_bwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
            got = gla.gla_bwd_layout(*t, gh, gw, scan, layout=layout, fwd_workspace=keep, workspace=room)
            got = [g if layout == 0 else g.transpose(1, 2) for g in got]
            for g, r in zip(got[:3], want[:3]):
                near(g, r)
            assert np.abs(got[3].cpu().numpy() - want[3]).max() <= TOL * 64 * size


@pytest.mark.parametrize("chunks", [288, 320, 399])
def test_one_long_sequence_and_its_states(chunks):
    """One sequence of 32 / 64 channels: whatever number of spans the forward call cut it into (up to 200 of them were two chunks long, more
    than the other kernels chain themselves), the backward call that takes its states finds local ones."""
    from oracle import gla_oracle
    dk, dv, gh, gw = 32, 64, chunks, 64
    d = gi.make_inputs(1, 1, gh * gw, dk, dv, "bf16", seed=chunks, z_mean=1.5)
    t = upload(d, "q", "k", "v", "log_alpha")
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((1, 1, gh * gw, dv)).astype(np.float32)).bfloat16()
    want = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, 0)
    ws = torch.full((gla.gla_fwd_workspace_bytes(1, 1, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    gla.gla_fwd_ex(*t, gh, gw, 0, workspace=ws)
    for got, ref in zip(gla.gla_bwd(*t, w.cuda(), gh, gw, 0, fwd_workspace=ws)[:3], want[:3]):
        near(got, ref)


def test_phases_of_one_launch():
    """gla_fwd_timed: the phases that a call in one launch does not have take no time; those of a call in two passes do."""
    B, H, gh, gw, dk, dv = 1, 16, 40, 64, 36, 72
    t = upload(gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=2), "q", "k", "v", "log_alpha")
    ws = torch.empty(gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16), dtype=torch.uint8, device="cuda")
    out, fin = gla.gla_fwd_ex(*t, gh, gw, 0, workspace=ws)
    ms = gla.gla_fwd_timed(*t, gh, gw, 0, out, fin, ws, iters=3)
    assert ms[0] == 0 and ms[1] == 0 and 0 < ms[2] <= ms[3]
    try:
        gla.gla_set_option(gla.OPT_CARRY, gla.CARRY_KERNEL)
        ms = gla.gla_fwd_timed(*t, gh, gw, 0, out, fin, ws, iters=3)
    finally:
        gla.gla_set_option(gla.OPT_CARRY, gla.CARRY_AUTO)
    assert all(0 < m < ms[3] for m in ms[:3])


def test_replays_do_not_take_old_states():
    """A recorded call has one nonce for all replays: other inputs in the same buffers, and calls outside the graph on the same
    workspace, must not be answered from the states that the flags of an earlier replay stand for."""
    B, H, gh, gw, dk, dv = 2, 16, 45, 61, 36, 72
    sets = [[x.cuda() for x in upload(gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=s, z_mean=3.0), "q", "k", "v", "log_alpha")] for s in (1, 2)]
    ws = torch.empty(gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16), dtype=torch.uint8, device="cuda")
    want = [[y.clone() for y in gla.gla_fwd_ex(*x, gh, gw, 2, workspace=ws)] for x in sets]
    t = [x.clone() for x in sets[0]]
    out, fin = torch.empty_like(want[0][0]), torch.empty_like(want[0][1])
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        gla.gla_fwd_ex(*t, gh, gw, 2, out=out, final_state=fin, workspace=ws, stream=side)
    for i in (0, 1, 1, 0):
        for x, y in zip(t, sets[i]):
            x.copy_(y)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[i][0]) and torch.equal(fin, want[i][1]), i
        got = gla.gla_fwd_ex(*sets[1 - i], gh, gw, 2, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[1 - i][0])
    # one replay behind the other, so that the flags of the one before are there unless the call clears them
    for i in (0, 1, 0, 0, 1, 1, 0):
        for x, y in zip(t, sets[i]):
            x.copy_(y)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[i][0]) and torch.equal(fin, want[i][1]), i
