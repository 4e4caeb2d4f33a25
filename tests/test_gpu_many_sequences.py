"""More sequences than a wide kernel's work-groups may be launched for at once (HIP takes fewer than 2^32 threads along one
dimension): a block of sequences repeated, every repetition equal to the block's own call."""
import pytest

torch = pytest.importorskip("torch")

import paper_2405_18428_amd as gla

pytestmark = pytest.mark.gpu


def _block(H, T, dk, dv, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    q, k, v = (randn(1, H, T, d).bfloat16() for d in (dk, dk, dv))
    return q, k, v, torch.nn.functional.logsigmoid(randn(1, H, T, dk)) / 16, randn(1, H, T, dv).bfloat16()


def _same(got, ref, what):
    for b in range(0, got.shape[0], 1000):       # (in pieces: the comparison makes a tensor of its own)
        assert bool((got[b:b + 1000] == ref).all()), what


@pytest.fixture(autouse=True)
def _room():
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    yield
    torch.cuda.empty_cache()


def test_token_by_token():
    """22.5 million sequences of 33 steps: three waves a work-group would be 4.3e9 threads."""
    n, H, T = 22000, 1024, 33
    *x, _ = _block(H, T, 1, 1, 0)
    ref, fin = gla.gla_fwd_ex(*x, 3, 11)
    got, got_fin = gla.gla_fwd_ex(*(t.repeat(n, 1, 1, 1) for t in x), 3, 11)
    # (two waves where the block has three: the second round's chain of local states sums in another order)
    for b in range(0, n, 1000):
        assert float((got[b:b + 1000] - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        assert float((got_fin[b:b + 1000] - fin).abs().max()) <= 1e-5 * float(fin.abs().max())


@pytest.mark.parametrize("layout", [gla.LAYOUT_BHTD, gla.LAYOUT_BTHD])
def test_large_heads_one_batch_element(layout):
    """The same with all sequences in one batch element (heads are cut, not batch elements), an initial state, bf16 out."""
    H, n, T, dk, dv = 1024, 8200, 1, 44, 8
    q, k, v, la, _ = (t.transpose(1, 2).contiguous() if layout else t for t in _block(H, T, dk, dv, 2))
    s0 = torch.randn(1, H, dk, dv, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    kw = dict(layout=layout, out_dtype=torch.bfloat16)
    ref, fin = gla.gla_fwd_layout(q, k, v, la, 1, 1, 0, initial_state=s0, **kw)
    many = [t.repeat(1, 1, n, 1) if layout else t.repeat(1, n, 1, 1) for t in (q, k, v, la)]
    got, got_fin = gla.gla_fwd_layout(*many, 1, 1, 0, initial_state=s0.repeat(1, n, 1, 1), **kw)
    _same(got.view(n, 1, H, T, dv) if not layout else got.view(n, 1, T, H, dv), ref, "out")
    _same(got_fin.view(n, 1, H, dk, dv), fin, "state")


def test_large_heads():
    """8.4 million sequences of one step at 44 / 8 channels, forward and backward: eight waves a work-group would be
    4.3e9 threads, so there are two launches of each kernel."""
    n, H = 8200, 1024
    *x, dout = _block(H, 1, 44, 8, 1)
    refs = (*gla.gla_fwd_ex(*x, 1, 1), *gla.gla_bwd(*x, dout, 1, 1))
    many = [t.repeat(n, 1, 1, 1) for t in x]
    for name, got, ref in zip(("out", "state"), gla.gla_fwd_ex(*many, 1, 1), refs):
        _same(got, ref, name)
    for name, got, ref in zip(("dq", "dk", "dv", "dlog_alpha"), gla.gla_bwd(*many, dout.repeat(n, 1, 1, 1), 1, 1), refs[2:]):
        _same(got, ref, name)
