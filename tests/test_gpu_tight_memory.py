"""Calls under a device-memory cap: the faster forms of a sum take memory that
the plain ones do not, and what fits in the plain form is not refused."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def open_system(s):
    from paper_2603_10295_amd import ephw
    ctx = ephw.Context(0)
    return ctx, ephw.System.from_synth(ctx, s)


@pytest.mark.parametrize("prec,nw,na,nk", [(0, 4, 8, 8), (1, 16, 8, 4), (1, 4, 8, 1)])
def test_loss_backward_takes_no_more_for_its_partials(prec, nw, na, nk):
    """One Re at a time needed partials of q x Nm^2 x K chunks; all of them are to
    fit the buffers that the call has anyway (the last case: one Re)."""
    import torch
    from gpu_run import cplx_dtype, dev
    s = synth.make_system(nw, na, synth.box((9, 9, 9)), synth.box((2, 1, 1)), [nw, 40],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    from paper_2603_10295_amd import ephw
    ctx, h = open_system(s)
    k = synth.uniform_grid((nk, 1, 1))
    q = k[:min(nk, 4)]
    kqi = synth.grid_index_of_sum((nk, 1, 1))[:len(q)].copy()
    ks = ephw.KSet(h, dev(k), prec)
    dg, dk, dq = (torch.zeros(s.g.shape, dtype=cplx_dtype(prec), device="cuda:0"),
                  torch.zeros((nk, 3), dtype=torch.float64, device="cuda:0"),
                  torch.zeros((len(q), 3), dtype=torch.float64, device="cuda:0"))
    before = ctx.memory()[0]
    ephw.loss_backward(ks, dev(q), dev(kqi), dL_dg=dg, dL_dk=dk, dL_dq=dq)
    ctx.check()
    took = ctx.memory()[0] - before
    cs, nq, ne, nm, nw2 = (16 if prec == 0 else 8), len(q), s.ne, s.nm, nw * nw
    E = nm * nw2
    # every buffer but the partials, which get one Re's worth
    each = nq * nm * nm * cs
    assert took <= 4 * nq * ne * E * cs + 5 * nk * nq * E * cs + each + (2 << 20)
    ks.close()
    h.close()
    ctx.close()


def test_partials_one_re_at_a_time():
    """The form of a unit whose other buffers hold no partial: 24 modes, 4 bands,
    one k.  Modes and bands are not degenerate."""
    import oracle.adjoint
    import torch
    from gpu_run import dev
    from paper_2603_10295_amd import ephw
    s = synth.make_system(4, 8, synth.box((3, 2, 1)), synth.box((2, 2, 1)), [4, 41])
    k = np.zeros((1, 3))
    ref = oracle.adjoint.loss_and_grads(s, k, k, 11)
    ctx, h = open_system(s)
    ks = ephw.KSet(h, dev(k), 0)
    dg = torch.zeros(s.g.shape, dtype=torch.complex128, device="cuda:0")
    dk, dq = torch.zeros((1, 3), dtype=torch.float64, device="cuda:0"), torch.zeros((1, 3), dtype=torch.float64, device="cuda:0")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    ephw.loss_backward(ks, dev(k), dev(np.zeros((1, 1), dtype=np.int32)), loss_seed=11, loss=loss, dL_dg=dg, dL_dk=dk, dL_dq=dq)
    ctx.check()
    for got, name in zip((loss, dg, dk, dq), ("loss", "dg", "dk", "dq")):
        got, want = got.cpu().numpy(), np.asarray(ref[name])
        assert np.abs(got.reshape(-1) - want.reshape(-1)).max() <= 1e-9 * np.abs(want).max()
    ks.close()
    h.close()
    ctx.close()


def test_compensated_sets_hold_one_copy_of_their_phases():
    from gpu_run import dev
    from paper_2603_10295_amd import ephw
    s = synth.make_system(4, 1, synth.box((9, 9, 9)), synth.box((1, 1, 1)), [4, 44], g_dtype=np.complex64)
    ctx, h = open_system(s)
    k = dev(np.random.default_rng(1).random((600, 3)))
    ks = ephw.KSet(h, k, ephw.FP32_COMP)
    held = ctx.memory()[0]
    ks.close()
    held -= ctx.memory()[0]
    assert held <= 600 * (24 + s.ne * 8 + len(s.r_h) * 16 + 4 * 8 + 16 * 24) + 6 * 256
    h.close()
    ctx.close()
