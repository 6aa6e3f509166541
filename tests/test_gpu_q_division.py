"""g of degenerate bands at interpolated k+q, where the states are the
eigensolver's choice: the same however the q list is divided over calls and
batches."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nw", [6, 7, 11, 16, 20])
def test_q_divided(prec, nw):
    import torch
    from gpu_run import Runner, cplx_dtype, dev
    from paper_2603_10295_amd import ephw
    run = Runner()
    s = synth.make_system(nw, 1, synth.box((3, 3, 1)), synth.box((2, 1, 1)), [nw, 9],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    rng = np.random.default_rng(nw)
    # H(k) = F(k) M, the eigenvalues of M in equal pairs
    z = np.linalg.qr(rng.standard_normal((nw, nw)) + 1j * rng.standard_normal((nw, nw)))[0]
    m = (z * (1.0 + np.arange(nw) // 2)) @ z.conj().T
    paired = (s.r_h[None] == -s.r_h[:, None]).all(-1).any(1)
    f = np.exp(-(s.r_h ** 2).sum(1)) * paired
    s = dataclasses.replace(s, h_r=f[:, None, None] * (0.5 * (m + m.conj().T)))
    nk, nq = 2 + 4000000 // (9 * nw ** 3), 9
    k, q = dev(rng.random((nk, 3))), dev(rng.random((nq, 3)))
    h = run.system(s)
    ks = ephw.KSet(h, k, prec)
    g = torch.empty((4, nq, nk, s.nm, nw, nw), dtype=cplx_dtype(prec), device="cuda:0")
    ephw.interpolate(ks, q, g_out=g[0])
    for j in range(nq):
        ephw.interpolate(ks, q[j:j + 1], g_out=g[1, j:j + 1])
    h.set_q_batch(2)
    ephw.interpolate(ks, q, g_out=g[2])
    h.set_q_batch(1)
    ephw.interpolate_noalloc(ks, q, g_out=g[3])
    run.ctx.check()
    top = float(g[0].abs().max())
    for i in (1, 2, 3):
        assert float((g[i] - g[0]).abs().max()) <= (1e-12 if prec == 0 else 1e-5) * top
    ks.close()
    h.close()
