"""ephw_interpolate_noalloc in a captured graph, in the forms of its sums and
eigensolves: every replay, with new q and eager work in between, against the
eager call."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nw,na,nk,capped", [
    (1, 8, 2, 600, False),     # packed, fused; tridiagonal k+q of order 8
    (1, 4, 2, 600, True),      # packed with the phases packed by the call, W stored
    (1, 4, 22, 40, False),     # D(q) of order 66: tridiagonal, then Jacobi where degenerate
    (0, 17, 1, 40, False),
    (2, 5, 1, 80, False),
])
def test_replays(prec, nw, na, nk, capped):
    import torch
    from gpu_run import cplx_dtype, dev
    from paper_2603_10295_amd import ephw
    s = synth.make_system(nw, na, synth.box((4, 4, 4)), synth.box((2, 2, 1)), [nw, 50],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    ctx = ephw.Context(0)
    h = ephw.System.from_synth(ctx, s)
    if capped:
        ctx.set_limits(max_device_bytes=1 << 30)
    rng = np.random.default_rng(nk)
    ks = ephw.KSet(h, dev(rng.random((nk, 3))), prec)
    q = dev(rng.random((3, 3)))
    out, ref = (torch.empty((3, nk, s.nm, nw, nw), dtype=cplx_dtype(prec), device="cuda:0") for _ in range(2))
    ephw.interpolate_noalloc(ks, q, g_out=out)      # kernels loaded before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ephw.interpolate_noalloc(ks, q, g_out=out)
    for i in range(4):
        q.copy_(dev(rng.random((3, 3)) if i != 2 else np.zeros((3, 3))))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        ephw.interpolate_noalloc(ks, q, g_out=ref)
        ctx.check()
        assert bool(torch.isfinite(torch.view_as_real(ref)).all()) and torch.equal(out, ref)
    ks.close()
    h.close()
    ctx.close()


def test_a_limit_raised_after_the_capture_counts():
    import torch
    from gpu_run import dev
    from paper_2603_10295_amd import ephw
    s = synth.make_system(4, 22, synth.box((2, 2, 1)), synth.box((2, 2, 1)), [4, 51], g_dtype=np.complex64)
    ctx = ephw.Context(0)
    h = ephw.System.from_synth(ctx, s)
    ks = ephw.KSet(h, dev(np.random.default_rng(1).random((5, 3))), 1)
    q = dev(np.random.default_rng(2).random((3, 3)))
    out, ref = (torch.empty((3, 5, 66, 4, 4), dtype=torch.complex64, device="cuda:0") for _ in range(2))
    t = torch.empty((3, 5, 66), dtype=torch.float64, device="cuda:0")

    def call(g):
        ephw.interpolate_noalloc(ks, q, flags=ephw.OUT_G | ephw.OUT_BAND_SUM, g_out=g, band_sum=t)
    call(ref)
    ctx.check()
    ctx.set_limits(max_sweeps=3)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    ctx.set_limits(max_sweeps=40)
    for _ in range(3):
        out.zero_()
        graph.replay()
        ctx.check()
        assert torch.equal(out, ref)
    ctx.set_limits(max_sweeps=3)
    graph.replay()
    with pytest.raises(ephw.EphwError) as e:
        ctx.check()
    assert e.value.status == ephw.ENOCONV
    ks.close()
    h.close()
    ctx.close()
