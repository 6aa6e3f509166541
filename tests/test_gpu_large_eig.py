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
