"""The token-by-token engine where its work is cut: rounds of 64 to 256 scan steps, 8 or 16 steps per wave, 16 columns
per work-group, channel classes 32 / 40 / 64 (key axis) and 32 / 64 / 72 / 128 (value axis).  fp32 inputs against the
fp64 oracles; bar 1e-4 x RMS as for every fp32 call (the sums run over at most a few hundred terms of ordinary size:
about 1e-6)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2405_18428_amd as gla
from paper_2405_18428_amd import inputs as gi
from oracle import gla_oracle as orc
from oracle import gla_oracle_gates as og

pytestmark = pytest.mark.gpu
TOL = 1e-4

SIZES = [
    # grid, dk, dv: one step; a wave's steps +- 1; a round +- 1; several rounds
    ((1, 1), 1, 1), ((3, 5), 32, 16), ((1, 16), 31, 17), ((1, 17), 33, 15), ((1, 63), 40, 72), ((1, 65), 41, 73),
    ((1, 127), 64, 128), ((3, 43), 36, 72), ((15, 17), 32, 64), ((16, 16), 32, 64), ((1, 257), 20, 33),
    ((19, 31), 36, 72), ((23, 41), 64, 65),
]


def _err(got, ref, floor=0.0):
    ref = np.asarray(ref, dtype=np.float64)
    rms = max(float(np.sqrt(np.mean(ref * ref))), floor)
    return float(np.abs(got.cpu().numpy().astype(np.float64) - ref).max() / max(rms, 1e-300))


@pytest.fixture(autouse=True)
def _plan():
    yield
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, 0)


@pytest.mark.parametrize("cps", [0, 1])
@pytest.mark.parametrize("grid,dk,dv", SIZES)
def test_edges(grid, dk, dv, cps):
    gh, gw = grid
    gla.gla_set_option(gla.OPT_CHUNKS_PER_SPAN, cps)
    d = gi.make_gate_inputs(2, 2, gh * gw, dk, dv, "f32", seed=gh * gw + dk)
    d["w"] = np.random.Generator(np.random.PCG64(9)).standard_normal(d["v"].shape, dtype=np.float32)
    q, k, v, la, lb, w = (torch.from_numpy(d[n]).cuda() for n in ("q", "k", "v", "log_alpha", "log_beta", "w"))
    host = [d[n] for n in ("q", "k", "v", "log_alpha")]
    for scan in (0, 3):
        out, fin = gla.gla_fwd_ex(q, k, v, la, gh, gw, scan)
        for got, ref in zip((out, fin), orc.gla_fwd(*host, gh, gw, scan)):
            assert _err(got, ref) < TOL
        out, fin = gla.gla_fwd_gates(q, k, v, la, lb, gh, gw, scan)
        for got, ref in zip((out, fin), og.gla_fwd_gates(*host, d["log_beta"], gh, gw, scan)):
            assert _err(got, ref) < TOL
        rms = lambda x: float(np.sqrt(np.mean(np.square(x, dtype=np.float64))))  # noqa: E731
        ref = orc.gla_bwd(*host, d["w"], gh, gw, scan)
        floors = [0, 0, 0, rms(d["q"] * ref[0])]      # (the gate gradients' terms can cancel altogether)
        for got, r, f in zip(gla.gla_bwd(q, k, v, la, w, gh, gw, scan), ref, floors):
            assert _err(got, r, f) < TOL
        ref = og.gla_bwd_gates(*host, d["log_beta"], d["w"], gh, gw, scan)
        floors = [0, 0, 0, rms(d["q"] * ref[0]), rms(d["v"] * ref[2])]
        for got, r, f in zip(gla.gla_bwd_gates(q, k, v, la, lb, w, gh, gw, scan), ref, floors):
            assert _err(got, r, f) < TOL


@pytest.mark.parametrize("B,H,grid,dk,dv", [
    # on both sides of the bounds up to which one thread per column walks a sequence of a few steps
    (1, 2, (1, 1), 36, 72), (1, 2, (2, 1), 32, 49), (1, 2, (1, 2), 33, 33), (1, 2, (1, 3), 36, 72), (32, 16, (2, 2), 64, 128),
    (32, 16, (1, 3), 31, 50), (32, 16, (1, 5), 36, 72), (64, 16, (2, 3), 36, 72), (64, 16, (1, 7), 40, 80)])
def test_few_steps(B, H, grid, dk, dv):
    gh, gw = grid
    T = gh * gw
    d = gi.make_gate_inputs(B, H, T, dk, dv, "f32", seed=T + dk)
    init = np.random.Generator(np.random.PCG64(8)).standard_normal((B, H, dk, dv), dtype=np.float32)
    host = [d[n] for n in ("q", "k", "v", "log_alpha")]
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    x, lb, s0 = [up(t) for t in host], up(d["log_beta"]), up(init)
    for scan in (0, 3):
        ref = orc.gla_fwd(*host, gh, gw, scan, initial_state=init)
        for got, r in zip(gla.gla_fwd_layout(*x, gh, gw, scan, initial_state=s0), ref):
            assert _err(got, r) < TOL
        bthd = [up(t.transpose(0, 2, 1, 3)) for t in host]
        out, fin = gla.gla_fwd_layout(*bthd, gh, gw, scan, layout=gla.LAYOUT_BTHD, initial_state=s0, out_dtype=torch.bfloat16)
        assert _err(out.float().transpose(1, 2), ref[0]) < 0.05 and _err(fin, ref[1]) < TOL    # (bf16: 2^-9 of the largest)
        for got, r in zip(gla.gla_fwd_gates(*x, lb, gh, gw, scan, initial_state=s0),
                          og.gla_fwd_gates(*host, d["log_beta"], gh, gw, scan, initial_state=init)):
            assert _err(got, r) < TOL
    assert _err(gla.gla_fwd_multi(*x, gh, gw, scan_dirs=(0, 1, 2, 3)), orc.gla_fwd_multi(*host, gh, gw, (0, 1, 2, 3))) < TOL


def test_closed_gates_stay_exact():
    """alpha = 0 (log alpha = -inf) and gates far below any factorised range, at steps on both sides of a wave's cut."""
    d = gi.make_inputs(1, 2, 80, 32, 20, "f32", seed=3)
    d["log_alpha"][:, :, 15::16, :] = -np.inf
    d["log_alpha"][:, :, 20:24, ::2] = -90.0
    out, fin = gla.gla_fwd_ex(*(torch.from_numpy(d[n]).cuda() for n in ("q", "k", "v", "log_alpha")), 8, 10, 0)
    ro, rf = orc.gla_fwd(d["q"], d["k"], d["v"], d["log_alpha"], 8, 10, 0)
    assert _err(out, ro) < TOL and _err(fin, rf) < TOL
