"""The bf16 hi/lo kernels that keep a chunk's rows in registers, at the edges of what they cover: numbers of key channels
around the 16-channel units and the tail, value columns around the 16-column tiles, chunks that are one token long or one
short, one span and several, both memory orders, an initial state; heads of up to 32 / 64 channels, which stay on the kernels that
stage rows through LDS, at the same edges.

Tolerance: the split operands carry 16 bits, so a product is off by at most 4 * 2^-17 of itself and an output, whose largest
value is about six times its RMS, by 2e-4 of the RMS; a bf16 store adds at most half a unit of its eighth bit, 2^-8 of the largest value."""
import numpy as np
import pytest
import torch

import paper_2405_18428_amd as gla
from paper_2405_18428_amd import inputs as gi

pytestmark = pytest.mark.gpu
TOL = 2e-4


@pytest.fixture(autouse=True)
def defaults():
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_MFMA)
    yield
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, 0)


def upload(d, name):
    return torch.from_numpy(d[name + "_bits"].view(np.int16)).cuda().view(torch.bfloat16)


@pytest.mark.parametrize("dk,dv", [(4, 8), (16, 64), (20, 24), (32, 64), (28, 72), (36, 8), (36, 72), (36, 80)])
@pytest.mark.parametrize("gh,gw", [(1, 1), (7, 9), (8, 8), (5, 13), (16, 16), (17, 19), (9, 50)])
def test_edges(dk, dv, gh, gw):
    from oracle import gla_oracle
    B, H, T = 2, 3, gh * gw
    d = gi.make_inputs(B, H, T, dk, dv, "bf16", seed=dk + dv)
    s0 = np.random.default_rng(5).standard_normal((B, H, dk, dv)).astype(np.float32)
    for cps, scan, layout, out_dtype in ((0, 0, 0, torch.float32), (1, 3, 1, torch.float32), (2, 2, 0, torch.bfloat16),
                                         (3, 1, 1, torch.float32)):
        gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
        ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, scan, initial_state=s0)
        t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda()]
        if layout == 1:
            t = [x.transpose(1, 2).contiguous() for x in t]
        out, fin = gla.gla_fwd_layout(*t, gh, gw, scan, layout=layout, initial_state=torch.from_numpy(s0).cuda(),
                                      out_dtype=out_dtype)
        got = out.float().cpu().numpy() if layout == 0 else out.float().transpose(1, 2).cpu().numpy()
        rms = np.sqrt(np.mean(ref ** 2))
        tol = TOL * max(1.0, np.abs(ref).max() / rms / 6) + (2.0 ** -8 * np.abs(ref).max() / rms if out_dtype == torch.bfloat16 else 0.0)
        assert np.abs(got - ref).max() / rms <= tol, (cps, scan, layout)
        assert np.abs(fin.cpu().numpy() - ref_fin).max() / np.sqrt(np.mean(ref_fin ** 2)) <= TOL, (cps, scan, layout)


@pytest.mark.parametrize("dk,dv", [(36, 8), (36, 72), (36, 80), (20, 72)])
@pytest.mark.parametrize("B,gh,gw", [(1, 1, 1), (1, 7, 9), (1, 8, 8), (1, 5, 13), (1, 17, 19), (1, 9, 50), (86, 5, 13)])
def test_walk_edges(dk, dv, B, gh, gw):
    """The backward walks at the same edges, one span and several, both memory orders, and at 258 sequences, where the
    older kernels take them.  The gate gradient is a sum over up to T steps of terms q dq - k dk, each off by at most TOL of
    their size: sqrt(T) TOL of it, whatever cancels."""
    from oracle import gla_oracle
    H, T = 3, gh * gw
    d = gi.make_inputs(B, H, T, dk, dv, "bf16", seed=dk + dv + 1)
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, T, dv)).astype(np.float32)).bfloat16()
    for cps, scan, layout in ((0, 0, 0), (1, 3, 1), (2, 2, 0), (3, 1, 0)):
        gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
        ref = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, scan)
        t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda(), w.cuda()]
        if layout == 1:
            t = [x.transpose(1, 2).contiguous() for x in t]
        got = gla.gla_bwd_layout(*t, gh, gw, scan, layout=layout)
        got = [(g if layout == 0 else g.transpose(1, 2)).cpu().numpy() for g in got]
        for g, r in zip(got[:3], ref[:3]):
            rms = np.sqrt(np.mean(r ** 2))
            assert np.abs(g - r).max() / rms <= TOL * max(1.0, np.abs(r).max() / rms / 6), (cps, scan, layout)
        size = max(np.sqrt(np.mean((d["q"].astype(np.float64) * ref[0]) ** 2)), np.sqrt(np.mean(ref[3] ** 2)))
        assert np.abs(got[3] - ref[3]).max() <= TOL * 6 * np.sqrt(T) * size, (cps, scan, layout)


def test_large_call():
    """3024 chunks: a column scan of these heads leaves the fp16 kernels for these, whose accuracy it then has."""
    from oracle import gla_oracle
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    B, H, gh, gw, dk, dv = 3, 16, 63, 64, 36, 72
    d = gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=3)
    ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, 2)
    t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda()]
    out, fin = gla.gla_fwd_layout(*t, gh, gw, 2, out_dtype=torch.float32)
    rms = np.sqrt(np.mean(ref ** 2))
    assert np.abs(out.cpu().numpy() - ref).max() / rms <= TOL * max(1.0, np.abs(ref).max() / rms / 6)
    assert np.abs(fin.cpu().numpy() - ref_fin).max() / np.sqrt(np.mean(ref_fin ** 2)) <= TOL


@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("B,gh,gw,scans", [(2, 64, 64, (0, 1)), (2, 64, 64, (2,)), (1, 112, 112, (0, 3)), (3, 63, 64, (2,)), (3, 63, 64, (0, 1))])
def test_reuse_takes_the_plan_of_the_forward_call(dk, dv, B, gh, gw, scans):
    """Span states of a forward call (several scan orders: of the last one) give the gradients that a call of its own states
    gives, also where the kernels that wrote them have span plans of their own; two sums over other spans, 2 TOL."""
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    H, T = 16 if gh < 100 else 6, gh * gw
    d = gi.make_inputs(B, H, T, dk, dv, "bf16", seed=4)
    t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda()]
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, T, dv)).astype(np.float32)).bfloat16().cuda()
    ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, T, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    if len(scans) == 1:
        gla.gla_fwd_layout(*t, gh, gw, scans[0], workspace=ws)
    else:
        gla.gla_fwd_multi(*t, gh, gw, scan_dirs=scans, workspace=ws)
    ref = gla.gla_bwd(*t, w, gh, gw, scans[-1])
    got = gla.gla_bwd(*t, w, gh, gw, scans[-1], fwd_workspace=ws)
    # a plain call's states may come from the fp16 kernels, whose operands carry 11 bits where the hi/lo pairs carry 16
    tol = 2 * TOL if len(scans) > 1 else 32 * TOL
    for g, r in zip(got[:3], ref[:3]):
        assert float((g - r).abs().max() / r.square().mean().sqrt()) <= tol * max(1.0, float(r.abs().max() / r.square().mean().sqrt()) / 6)


@pytest.mark.parametrize("engine", [gla.ENGINE_AUTO, gla.ENGINE_MFMA])
@pytest.mark.parametrize("step", [0, 5, 20, 31, 40, 63])
def test_gate_of_exactly_zero(engine, step):
    """log_alpha = -inf on some channels at one step of a chunk, and a step whose pre-activation is as low: the limits of the
    engines do not cover it, but no output is lost to NaN, and six chunks later, where the steps of that chunk have decayed to
    less than TOL, the results are right again."""
    from oracle import gla_oracle
    gla.gla_set_option(gla.OPT_ENGINE, engine)
    B, H, gh, gw, dk, dv = 1, 3, 16, 48, 36, 72
    T, at = gh * gw, 2 * 64 + step
    d = gi.make_inputs(B, H, T, dk, dv, "bf16", seed=7)
    d["log_alpha"][:, :, at, [0, 5, 17, 33, 35]] = -np.inf
    t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda()]
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, T, dv)).astype(np.float32)).bfloat16()
    z = torch.from_numpy(np.random.default_rng(8).standard_normal((B, H, T, dk)).astype(np.float32))
    z[:, :, at, [0, 5, 17, 33, 35]] = -3e38
    for cps in (0, 3, 12):
        gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
        ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, 0)
        out, fin = gla.gla_fwd_layout(*t, gh, gw, 0, out_dtype=torch.float32)
        out, fin = out.cpu().numpy(), fin.cpu().numpy()
        assert np.isfinite(out).all() and np.isfinite(fin).all()
        rms = np.sqrt(np.mean(ref ** 2))
        assert np.abs(out - ref)[:, :, 9 * 64:].max() / rms <= TOL * max(1.0, np.abs(ref).max() / rms / 6)
        assert np.abs(fin - ref_fin).max() / np.sqrt(np.mean(ref_fin ** 2)) <= TOL
        for g in gla.gla_bwd(*t, w.cuda(), gh, gw, 0):
            assert bool(torch.isfinite(g).all())
        fused, fin = gla.gla_fwd_fused(*t[:3], z.bfloat16().cuda(), 16.0, gh, gw, 0)
        assert bool(torch.isfinite(fused).all()) and bool(torch.isfinite(fin).all())


@pytest.mark.parametrize("B,chunks", [(16, 16), (17, 16), (20, 8), (24, 25), (40, 64)])
def test_many_sequences_are_walked_in_one_pass(B, chunks):
    """Calls of more sequences than compute units: the state pass that several spans a sequence would need costs more than what
    they would gain (272 sequences of 16 chunks 65 us in one span, 75 in three), so nothing is left in the workspace."""
    H, gh, gw, dk, dv = 16, chunks, 64, 36, 72
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(B, H, gh * gw, d, generator=g, device="cuda").bfloat16() for d in (dk, dk, dv))
    la = torch.full((B, H, gh * gw, dk), -0.05, device="cuda")
    ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    gla.gla_fwd_layout(q, k, v, la, gh, gw, 0, workspace=ws)
    written = int((ws != 0xFF).sum())
    assert written == 0
    gla.gla_fwd_fused(q, k, v, la.bfloat16(), 16.0, gh, gw, 0, r_pre=v, workspace=ws)
    written = int((ws != 0xFF).sum())
    assert written == 0


@pytest.mark.parametrize("cps", [1, 2, 3, 4, 5, 9, 10])
@pytest.mark.parametrize("scan,layout", [(1, 0), (2, 0), (0, 1), (3, 1)])
def test_lengths_of_spans(cps, scan, layout):
    """Four spans (the last one ragged) of the lengths between which the passes change from the kernels that stage rows through
    LDS to those that hold them in registers, forwards and backwards, also from the forward call's states."""
    from oracle import gla_oracle
    B, H, gh, gw, dk, dv = 1, 2, 4 * cps, 61, 36, 72
    T = gh * gw
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
    d = gi.make_inputs(B, H, T, dk, dv, "bf16", seed=cps)
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, H, T, dv)).astype(np.float32)).bfloat16()
    ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, scan)
    grad = gla_oracle.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w.float().numpy(), gh, gw, scan)
    t = [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda(), w.cuda()]
    if layout == 1:
        t = [x.transpose(1, 2).contiguous() for x in t]
    ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, T, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    out, fin = gla.gla_fwd_layout(*t[:4], gh, gw, scan, layout=layout, out_dtype=torch.float32, workspace=ws)
    back = (lambda x: x.cpu().numpy()) if layout == 0 else (lambda x: x.transpose(1, 2).cpu().numpy())

    def near(got, want):
        rms = np.sqrt(np.mean(want ** 2))
        assert np.abs(got - want).max() / rms <= TOL * max(1.0, np.abs(want).max() / rms / 6)

    near(back(out), ref)
    near(fin.cpu().numpy(), ref_fin)
    # (the gate gradient as in test_walk_edges)
    size = max(np.sqrt(np.mean((d["q"].astype(np.float64) * grad[0]) ** 2)), np.sqrt(np.mean(grad[3] ** 2)))
    for keep in (None, ws):
        got = [back(g) for g in gla.gla_bwd_layout(*t, gh, gw, scan, layout=layout, fwd_workspace=keep)]
        for g, r in zip(got[:3], grad[:3]):
            near(g, r)
        assert np.abs(got[3] - grad[3]).max() <= TOL * 6 * np.sqrt(T) * size


@pytest.mark.parametrize("B", [16, 17, 33])
@pytest.mark.parametrize("chunks", [1, 2, 3, 6, 7])
def test_short_sequences_with_the_heads_inside(B, chunks):
    """[B,T,H,d] rows of 256, 272 and 528 sequences of one span, on either side of the lengths that stay with the kernels that
    stage rows through LDS: every sequence as in a call of its own, which is on the others."""
    H, gh, gw, dk, dv = 16, chunks, 63, 36, 72
    g = torch.Generator(device="cuda").manual_seed(chunks)
    q, k, v = (torch.randn(B, gh * gw, H, d, generator=g, device="cuda").bfloat16() for d in (dk, dk, dv))
    la = torch.nn.functional.logsigmoid(torch.randn(B, gh * gw, H, dk, generator=g, device="cuda")) / 16
    s0 = torch.randn(B, H, dk, dv, generator=g, device="cuda")
    for scan in (0, 3):
        out, fin = gla.gla_fwd_layout(q, k, v, la, gh, gw, scan, layout=1, initial_state=s0, out_dtype=torch.float32)
        for b in (0, B // 2, B - 1):
            one, last = gla.gla_fwd_layout(*(x[b:b + 1] for x in (q, k, v, la)), gh, gw, scan, layout=1,
                                           initial_state=s0[b:b + 1], out_dtype=torch.float32)
            for x, y in ((out[b:b + 1], one), (fin[b:b + 1], last)):
                rms = float(y.square().mean().sqrt())
                assert float((x - y).abs().max()) / rms <= 2 * TOL * max(1.0, float(y.abs().max()) / rms / 6), (b, scan)


@pytest.mark.parametrize("scan,out_dtype", [(0, torch.float32), (3, torch.bfloat16)])
def test_large_call_with_the_heads_inside(scan, out_dtype):
    """3024 chunks of [B,T,H,d] rows leave the fp16 kernels for these in either kind of scan, and the backward call finds the
    span states on the plan that this choice gives."""
    from oracle import gla_oracle
    gla.gla_set_option(gla.OPT_ENGINE, gla.ENGINE_AUTO)
    B, H, gh, gw, dk, dv = 3, 16, 63, 64, 36, 72
    d = gi.make_inputs(B, H, gh * gw, dk, dv, "bf16", seed=3)
    ref, ref_fin = gla_oracle.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], gh, gw, scan)
    t = [x.transpose(1, 2).contiguous() for x in [upload(d, n) for n in ("q", "k", "v")] + [torch.from_numpy(d["log_alpha"]).cuda()]]
    ws = torch.full((gla.gla_fwd_workspace_bytes(B, H, gh * gw, dk, dv, gla.DT_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    out, fin = gla.gla_fwd_layout(*t, gh, gw, scan, layout=1, out_dtype=out_dtype, workspace=ws)
    rms = np.sqrt(np.mean(ref ** 2))
    tol = TOL * max(1.0, np.abs(ref).max() / rms / 6) + (2.0 ** -8 * np.abs(ref).max() / rms if out_dtype == torch.bfloat16 else 0.0)
    assert np.abs(out.float().transpose(1, 2).cpu().numpy() - ref).max() / rms <= tol
    assert np.abs(fin.cpu().numpy() - ref_fin).max() / np.sqrt(np.mean(ref_fin ** 2)) <= TOL
    w = torch.from_numpy(np.random.default_rng(9).standard_normal((B, gh * gw, H, dv)).astype(np.float32)).bfloat16().cuda()
    own = gla.gla_bwd_layout(*t, w, gh, gw, scan, layout=1)
    got = gla.gla_bwd_layout(*t, w, gh, gw, scan, layout=1, fwd_workspace=ws)
    for g, r in zip(got[:3], own[:3]):      # (two sums over other spans)
        assert float((g - r).abs().max() / r.square().mean().sqrt()) <= 2 * TOL * max(1.0, float(r.abs().max() / r.square().mean().sqrt()) / 6)
