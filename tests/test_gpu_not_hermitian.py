"""H(R) and C(R) whose partner at -R is missing or not its conjugate transpose
(hand-written or truncated files): every call treats the resulting matrices
alike.  Up to order 32 the solvers take the upper triangle; above, a matrix that
is not Hermitian does not converge."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nw", [8, 11, 17, 24, 32])
def test_bands_at_kq_are_those_of_the_points(prec, nw):
    import torch
    from gpu_run import Runner
    from paper_2603_10295_amd import ephw
    run = Runner()
    s = synth.make_system(nw, 1, synth.box((3, 2, 1)), synth.box((2, 1, 1)), [nw, 6],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    rng = np.random.default_rng(nw)
    s = dataclasses.replace(s, h_r=s.h_r + 1e-3 * rng.standard_normal(s.h_r.shape))
    nk = 4000000 // (5 * nw ** 3) + 2
    k, q = rng.random((nk, 3)), rng.random((5, 3))
    h = run.system(s)
    got = run.interpolate(h, k, q, prec, flags=ephw.OUT_G)["eps_kq"]
    want, _ = run.bands(h, (q[:, None] + k).reshape(-1, 3))
    assert np.abs(got.reshape(-1, nw) - want).max() <= 1e-13 * nw * np.abs(want).max()


@pytest.mark.parametrize("nw,na", [(2, 22), (33, 22)])
def test_large_modes_that_do_not_converge(nw, na):
    import torch
    from gpu_run import Runner
    from paper_2603_10295_amd import ephw
    run = Runner()
    s = synth.make_system(nw, na, synth.box((2, 1, 1)), synth.box((2, 1, 1)), [nw, 7], g_dtype=np.complex64)
    s = dataclasses.replace(s, c_r=s.c_r + 1e-9 * np.random.default_rng(1).standard_normal(s.c_r.shape))
    h = run.system(s)
    k = np.array([[0, 0, 0], [0.5, 0, 0]])
    for call in (lambda: run.phonons(h, k),
                 lambda: run.interpolate(h, k, k, 1, kq_index=np.array([[0, 1], [1, 0]], dtype=np.int32),
                                         flags=ephw.OUT_G)):
        with pytest.raises(ephw.EphwError) as e:
            call()
        assert e.value.status == ephw.ENOCONV
