"""The eigensolves above 32 at the edges of their kernels: the smallest order,
odd orders (a pair of every round lacks a player), rows that do not fill a
wavefront's share, more than 64 pairs, and the largest order; eigenvalues
against LAPACK, residual and orthogonality of the vectors."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [33, 34, 47, 127, 129, 130, 255, 256])
def test_orders(nw):
    from gpu_run import Runner
    run = Runner()
    s = synth.make_system(nw, 1, synth.box((3, 1, 1)), synth.box((1, 1, 1)), [nw, 5], with_g=True)
    k = np.array([[0.0, 0, 0], [0.13, 0, 0], [0.5, 0, 0]])
    eps, vec = run.bands(run.system(s), k)
    h = oracle.hamiltonian_k(s, k)
    for i in range(len(k)):
        # n rounding errors of 2^-53 each, per column, and the stopping norm 1e-14
        tol = (1e-14 + 4 * nw * 2.0 ** -53) * np.linalg.norm(h[i])
        assert np.abs(eps[i] - np.linalg.eigvalsh(h[i])).max() <= tol
        assert np.abs(h[i] @ vec[i] - vec[i] * eps[i]).max() <= tol
        assert np.abs(vec[i].conj().T @ vec[i] - np.eye(nw)).max() <= 8 * nw * 2.0 ** -53 + 1e-14
        top = np.take_along_axis(vec[i], np.abs(vec[i]).argmax(0)[None], 0)[0]
        assert np.all(top.real > 0) and np.abs(top.imag).max() <= 1e-15


@pytest.mark.parametrize("nw", [7, 8, 9, 11, 12, 13, 16, 17, 23, 24, 25, 31, 32])
def test_tridiagonal_orders(nw):
    """The k+q eigensolves of the calls whose rounding is free, at every padded
    order's edges, a last wavefront that is not full, and a block-diagonal
    H(k) (reflections and QL rotations that vanish) with a repeated
    eigenvalue: bands against LAPACK, g by block sums against the oracle."""
    import dataclasses
    from gpu_run import Runner
    from paper_2603_10295_amd import ephw
    run = Runner()
    s = synth.make_system(nw, 1, synth.box((3, 2, 1)), synth.box((2, 1, 1)), [nw, 6])
    rng = np.random.default_rng(nw)
    # up to order 16 it takes n^3 x matrices of 4 million
    nk = 7 if nw > 16 else 4000000 // (5 * nw ** 3) + 2
    k, q = rng.random((nk, 3)), rng.random((5, 3))
    h = s.h_r.copy()
    h[:, 0, :] = h[:, :, 0] = h[:, 4, :] = h[:, :, 4] = 0   # two uncoupled equal bands
    zero = np.flatnonzero(~s.r_h.any(1))[0]
    h[zero, 0, 0] = h[zero, 4, 4] = 0.7
    for hr in (s.h_r, h, 1e-160 * s.h_r, 0 * h):
        t = dataclasses.replace(s, h_r=hr)
        got = run.interpolate(run.system(t), k, q, 0, flags=ephw.OUT_G)
        ref = oracle.interpolate(t, k, q, return_all=True)
        scale = max(np.abs(ref["eps_kq"]).max(), 1e-300)
        assert np.abs(got["eps_kq"] - ref["eps_kq"]).max() <= (1e-14 + 8 * nw * 2.0 ** -53) * nw * scale
        if hr is s.h_r:
            a = oracle.block_sums(np.abs(got["g"]) ** 2, ref["eps_kq"], ref["eps_k"], ref["lam"])
            b = oracle.block_sums(np.abs(ref["ghat"]) ** 2, ref["eps_kq"], ref["eps_k"], ref["lam"])
            assert oracle.compare_block_sums(a, b)[0] <= 1e-10
        # the rotations stay unitary whatever the spectrum: the sum over all bands
        # (the V(k) in it come from the k-set's own solves, whose squares leave
        # the FP64 range at 1e-160: eigenvalues only there)
        if 0 < scale < 1e-150 and hr.any():
            continue
        ta = (np.abs(got["g"]) ** 2).sum((-2, -1))
        tb = (np.abs(ref["ghat"]) ** 2).sum((-2, -1))
        assert np.abs(ta - tb).max() <= 1e-12 * tb.max()


@pytest.mark.parametrize("na,nq", [(11, 256), (12, 257), (21, 260), (22, 3), (43, 4), (64, 4), (85, 4)])
def test_tridiagonal_phonons(na, nq):
    """D(q) of orders 33 to 255 in a call whose rounding is free: one or two
    row blocks and their edges, uncoupled equal modes (columns with nothing to
    reflect, QL that splits), all zero; frequencies against LAPACK, g by block
    sums against the oracle, and the sum over all modes, which is that of any
    unitary e."""
    import dataclasses
    from gpu_run import Runner
    from paper_2603_10295_amd import ephw
    run = Runner()
    s = synth.make_system(2 if na < 33 else 33, na, synth.box((2, 2, 1)), synth.box((3, 2, 1)), [na, 7])
    nm = 3 * na
    rng = np.random.default_rng(na)
    k, q, kqi = rng.random((3, 3)), rng.random((nq, 3)), None
    if na >= 33:                      # so many modes take Nw > 32, and that a k grid
        k = q = np.array([[0, 0, 0], [0.25, 0, 0], [0.5, 0, 0], [0.75, 0, 0]])
        kqi = ((np.arange(4)[:, None] + np.arange(4)) % 4).astype(np.int32)
    c = s.c_r.copy()
    c[:, 0, :] = c[:, :, 0] = c[:, 4, :] = c[:, :, 4] = 0
    zero = np.flatnonzero(~s.r_c.any(1))[0]
    c[zero, 0, 0] = c[zero, 4, 4] = 0.7
    for cr in (s.c_r, c, 0 * c):
        t = dataclasses.replace(s, c_r=cr)
        got = run.interpolate(run.system(t), k, q, 0, kq_index=kqi, flags=ephw.OUT_G)
        ref = oracle.interpolate(t, k, q, return_all=True)
        lam = np.sort(np.abs(ref["lam"]), -1)
        assert np.abs(np.sort(got["omega"] ** 2, -1) - lam).max() <= (1e-14 + 8 * nm * 2.0 ** -53) * nm * lam.max()
        if cr is s.c_r:
            a = oracle.block_sums(np.abs(got["g"]) ** 2, ref["eps_kq"], ref["eps_k"], ref["lam"])
            b = oracle.block_sums(np.abs(ref["ghat"]) ** 2, ref["eps_kq"], ref["eps_k"], ref["lam"])
            assert oracle.compare_block_sums(a, b)[0] <= 1e-10
        ta = (np.abs(got["g"]) ** 2).sum((-3, -2, -1))
        tb = (np.abs(ref["ghat"]) ** 2).sum((-3, -2, -1))
        assert np.abs(ta - tb).max() <= 1e-12 * tb.max()
