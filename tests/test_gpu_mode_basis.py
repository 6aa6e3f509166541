"""One basis of the modes in every call, also inside the degenerate blocks of
D(q), where an eigensolver is free to choose: the nu of g is that of
ephw_phonons in each precision and entry point, and the loss of one call is the
one whose gradient another call returns."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def degenerate_system(nw, na, prec, groups=3, mirror=False):
    """D(q) = F(q) M with every eigenvalue of M repeated `groups` times, or
    (mirror) none repeated, but every mode as large on one half of the atoms as on
    the other"""
    s = synth.make_system(nw, na, synth.box((4, 1, 1)), synth.box((2, 2, 1)), [nw, na],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    rng = np.random.default_rng(na)
    qm = np.linalg.qr(rng.standard_normal((s.nm, s.nm)))[0]
    if mirror:
        a, b = (x + x.T for x in rng.standard_normal((2, s.nm // 2, s.nm // 2)))
        m = np.block([[a, b], [b, a]])
    else:
        m = (qm * np.repeat(1.0 + np.arange(-(-s.nm // groups)), groups)[:s.nm]) @ qm.T
    paired = (s.r_c[None] == -s.r_c[:, None]).all(-1).any(1)
    f = np.exp(-(s.r_c ** 2).sum(1)) * paired
    return dataclasses.replace(s, c_r=f[:, None, None] * (0.5 * (m + m.T)), mass=np.full(na, 2.0))


def grid(nq):
    k = np.array([[i / 4, 0, 0] for i in range(4)])
    q = k[np.arange(nq) % 4]
    return k, q, ((np.arange(nq)[:, None] + np.arange(4)) % 4).astype(np.int32)


def reference(run, h, s, ks, q, kqi):
    """Eq. (7) in 64 bits with V(k) of the set and the modes of ephw_phonons"""
    import torch
    vec = torch.empty((4, s.nw, s.nw), dtype=torch.complex128, device="cuda:0")
    ks.bands(None, vec)
    v, (lam, _, e) = vec.cpu().numpy(), run.phonons(h, q)
    u = e / np.sqrt(np.repeat(s.mass, 3))[:, None]
    k = np.array([[i / 4, 0, 0] for i in range(4)])
    w = oracle.phases(q, s.r_p) @ s.g.astype(np.complex128).reshape(len(s.r_p), -1)
    w = w.reshape(len(q), len(s.r_e), -1).transpose(1, 0, 2).reshape(len(s.r_e), -1)
    w = (oracle.phases(k, s.r_e) @ w).reshape(4, len(q), s.nm, -1)
    w = np.matmul(u.transpose(0, 2, 1)[None], w).reshape(4, len(q), s.nm, s.nw, s.nw).swapaxes(0, 1)
    return np.matmul(np.matmul(v[kqi].conj().swapaxes(-1, -2)[:, :, None], w), v[None, :, None])


# every call that takes the sizes: pair lists and the static scratch have up to 32
# bands, pair lists no compensated sets
FORMS = [(how, prec, nw, na, nq)
         for nw, na, nq in [(4, 2, 9), (4, 6, 5), (1, 6, 2100), (4, 8, 5), (3, 10, 5), (3, 12, 260), (2, 22, 5), (33, 22, 3)]
         for prec in (0, 1, 2) for how in ("interpolate", "noalloc", "with_loss", "pairs")
         if not (nw > 32 and how in ("noalloc", "pairs")) and not (prec == 2 and how == "pairs")]


@pytest.mark.parametrize("how,prec,nw,na,nq", FORMS)
def test_modes_are_those_of_phonons(how, prec, nw, na, nq):
    import torch
    from gpu_run import Runner, cplx_dtype, dev
    from paper_2603_10295_amd import ephw
    run, s = Runner(), degenerate_system(nw, na, prec)
    k, q, kqi = grid(nq)
    h = run.system(s)
    ks = ephw.KSet(h, dev(k), prec)
    g = torch.empty((nq, 4, s.nm, nw, nw), dtype=cplx_dtype(prec), device="cuda:0")
    if how == "pairs":
        ephw.interpolate_pairs(ks, dev(q), ephw.PAIRS_BY_Q, 4 * np.arange(nq + 1), dev(np.tile(np.arange(4), nq).astype(np.int32)),
                               dev(kqi.reshape(-1)), flags=ephw.OUT_G, g_out=g.reshape(4 * nq, s.nm, nw, nw))
    else:
        loss = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        fn = ephw.interpolate_noalloc if how == "noalloc" else ephw.interpolate
        fn(ks, dev(q), kq_index=dev(kqi), flags=ephw.OUT_G | (ephw.OUT_LOSS if how == "with_loss" else 0), g_out=g,
           loss=loss)
    run.ctx.check()
    ref = reference(run, h, s, ks, q, kqi)
    # sums of at most 16 terms and rotations of at most nm and nw, a few roundings each
    tol = 1e-12 if prec == 0 else 1e-5
    assert np.abs(g.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    ks.close()
    h.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nw,na,nq", [(4, 6, 5), (1, 6, 2100), (4, 8, 5), (3, 10, 5), (3, 12, 260), (2, 22, 5), (33, 22, 3)])
def test_modes_with_equal_components(prec, nw, na, nq):
    """Modes even or odd under a mirror: no solver's last bits may choose the
    component that fixes the phase."""
    import torch
    from gpu_run import Runner, cplx_dtype, dev
    from paper_2603_10295_amd import ephw
    run, s = Runner(), degenerate_system(nw, na, prec, mirror=True)
    k, q, kqi = grid(nq)
    h = run.system(s)
    ks = ephw.KSet(h, dev(k), prec)
    g = torch.empty((nq, 4, s.nm, nw, nw), dtype=cplx_dtype(prec), device="cuda:0")
    ephw.interpolate(ks, dev(q), kq_index=dev(kqi), g_out=g)
    run.ctx.check()
    ref = reference(run, h, s, ks, q, kqi)
    # the modes' own error is a rounding over the gaps, here at least 1e-5 of the norm
    tol = 1e-9 if prec == 0 else 1e-5
    assert np.abs(g.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    ks.close()
    h.close()


@pytest.mark.parametrize("nw,na", [(4, 6), (4, 8), (3, 9), (33, 22)])
def test_loss_and_gradient_belong_together(nw, na):
    """FP64: L is quadratic in g, so central differences of the loss of
    ephw_interpolate along any direction equal the gradient's product with it."""
    import torch
    from gpu_run import Runner, dev
    from paper_2603_10295_amd import ephw
    run, s = Runner(), degenerate_system(nw, na, 0)
    k, q, kqi = grid(3)
    h = run.system(s)
    ks = ephw.KSet(h, dev(k), 0)
    g0 = dev(s.g)
    d = torch.randn(s.g.shape, dtype=torch.complex128, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(3))

    def loss(t):
        h.set_g(g0 + t * d)
        out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        ephw.interpolate(ks, dev(q), kq_index=dev(kqi), flags=ephw.OUT_LOSS, loss=out, loss_seed=5)
        run.ctx.check()
        return float(out.cpu()[0])
    numeric = (loss(0.5) - loss(-0.5))
    l0 = loss(0.0)
    back, dg = torch.zeros(1, dtype=torch.float64, device="cuda:0"), torch.zeros_like(g0)
    ephw.loss_backward(ks, dev(q), dev(kqi), loss_seed=5, loss=back, dL_dg=dg)
    run.ctx.check()
    assert abs(float(back.cpu()[0]) - l0) <= 1e-11 * l0
    slope = float((dg.conj() * d).real.sum().cpu())
    scale = float(torch.linalg.vector_norm(dg).cpu()) * float(torch.linalg.vector_norm(d).cpu())
    assert abs(numeric - slope) <= 1e-10 * scale
    ks.close()
    h.close()
