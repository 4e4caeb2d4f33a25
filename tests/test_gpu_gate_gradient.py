"""Gate gradients formed inside the reversed walk of the backward pass: span bounds of ragged sequences, slowly decaying
gates (the start of every span then carries most of the sum), and workspaces without room for what the walk for dq leaves
(a state pass of the reversed recurrence and the separate reverse-cumulative-sum kernels).  Bar 2e-2 x RMS as for every
bf16 call.  The two routes differ by the rounding of sums of T terms, at most T 2^-24 of their largest partial sum (about
1e-3 of the RMS here)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2405_18428_amd as gla
from paper_2405_18428_amd import inputs as gi
from oracle import gla_oracle as orc
from oracle import gla_oracle_gates as og

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.fixture(autouse=True)
def _plan():
    yield
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, 0)


def _err(got, ref, floor):
    rms = max(float(np.sqrt(np.mean(np.square(ref)))), floor)
    return float(np.abs(got.cpu().numpy().astype(np.float64) - ref).max() / rms)


@pytest.mark.parametrize("B,H,gh,gw,cps", [
    (1, 3, 1, 64, 1), (1, 3, 1, 65, 1), (1, 3, 5, 77, 2), (1, 3, 19, 31, 3), (1, 3, 16, 40, 2), (1, 3, 1, 1023, 5),
    # more than 256 work-groups, which the kernels of 4 waves walk: one wave for the row read and the outputs
    (6, 16, 5, 77, 1), (6, 16, 5, 77, 2), (9, 16, 3, 43, 1), (65, 4, 1, 61, 1)])
@pytest.mark.parametrize("dk,dv", [(36, 72), (32, 64)])
@pytest.mark.parametrize("z_mean", [0.0, 3.0])
def test_span_bounds(B, H, gh, gw, cps, dk, dv, z_mean):
    T = gh * gw
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
    d = gi.make_gate_inputs(B, H, T, dk, dv, "bf16", seed=T + dk, z_mean=z_mean)
    bits = gi.round_to_bf16_bits(np.random.Generator(np.random.PCG64(5)).standard_normal((B, H, T, dv), dtype=np.float32))
    w = gi.bf16_bits_to_f32(bits)
    up = lambda b: torch.from_numpy(b.view(np.int16)).cuda().view(torch.bfloat16)  # noqa: E731
    q, k, v = (up(d[n + "_bits"]) for n in "qkv")
    dw = up(bits)
    la, lb = (torch.from_numpy(d[n]).cuda() for n in ("log_alpha", "log_beta"))
    # the least a workspace may hold: the span states, and the totals of the reverse cumulative sums (256 steps each)
    totals = lambda width: (B * H * ((T + 255) // 256) * width * 4 + 255) // 256 * 256  # noqa: E731
    least = gla.gla_fwd_workspace_bytes(B, H, T, dk, dv) + totals(dk)
    least_gates = gla.gla_fwd_workspace_bytes(B, H, T, dk, dv) + totals(dv) + (B * H * T * dv * 4 + 255) // 256 * 256
    for scan in (0, 3):
        ref = orc.gla_bwd(d["q"], d["k"], d["v"], d["log_alpha"], w, gh, gw, scan)
        floor = float(np.sqrt(np.mean(np.square(d["q"] * ref[0]))))
        routes = []
        for room in (gla.gla_bwd_workspace_bytes(B, H, T, dk, dv), least):
            ws = torch.empty(room, dtype=torch.uint8, device="cuda")
            got = gla.gla_bwd(q, k, v, la, dw, gh, gw, scan, workspace=ws)
            assert max(_err(g, r, f) for g, r, f in zip(got, ref, (0, 0, 0, floor))) <= TOL
            routes.append(got[3].cpu().numpy().astype(np.float64))
        assert _err(torch.from_numpy(routes[0]), routes[1], floor) <= 2e-3
        ref = og.gla_bwd_gates(d["q"], d["k"], d["v"], d["log_alpha"], d["log_beta"], w, gh, gw, scan)
        floors = (0, 0, 0, float(np.sqrt(np.mean(np.square(d["q"] * ref[0])))), float(np.sqrt(np.mean(np.square(d["v"] * ref[2])))))
        routes = []
        for room in (gla.gla_bwd_gates_workspace_bytes(B, H, T, dk, dv), least_gates):
            ws = torch.empty(room, dtype=torch.uint8, device="cuda")
            got = gla.gla_bwd_gates(q, k, v, la, lb, dw, gh, gw, scan, workspace=ws)
            assert max(_err(g, r, f) for g, r, f in zip(got, ref, floors)) <= TOL
            routes.append([g.cpu().numpy().astype(np.float64) for g in got[3:]])
        for a, b, f in zip(*routes, floors[3:]):
            assert _err(torch.from_numpy(a), b, f) <= 2e-3


@pytest.mark.parametrize("zeros", [3, 9, 20])
def test_two_sided_chain_behind_a_zero_tail(zeros):
    """k = 0 over the last chunks: the state entering a span behind them is the decayed sum of many earlier spans, all of
    them added up however far the zeros have decayed them (one chunk per span, chained by the output pass); the carry
    kernel, which has no cut-off, as second opinion.  Bar 1e-4 x RMS, twice the hi/lo kernels' error."""
    B, H, gh, gw, dk, dv = 1, 2, 64, 64, 36, 72
    d = gi.make_gate_inputs(B, H, gh * gw, dk, dv, "bf16", seed=zeros, z_mean=1.5)
    d["k"][:, :, (64 - zeros) * 64:] = 0.0
    d["k_bits"] = gi.round_to_bf16_bits(d["k"])
    q, k, v = (torch.from_numpy(d[n + "_bits"].view(np.int16)).cuda().view(torch.bfloat16) for n in "qkv")
    la, lb = (torch.from_numpy(d[n]).cuda() for n in ("log_alpha", "log_beta"))
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, 1)
    ref, ref_fin = og.gla_fwd_gates(d["q"], d["k"], d["v"], d["log_alpha"], d["log_beta"], gh, gw, 0)
    try:
        for carry in (gla.CARRY_KERNEL, gla.CARRY_IN_OUTPUT_PASS):
            gla.gla_set_option(gla.OPT_CARRY, carry)
            out, fin = gla.gla_fwd_gates(q, k, v, la, lb, gh, gw, 0)
            assert _err(out, ref, 0) <= 1e-4 and _err(fin, ref_fin, 0) <= 1e-4, carry
    finally:
        gla.gla_set_option(gla.OPT_CARRY, gla.CARRY_AUTO)
