"""Both sides of the rules that choose a kernel by the number of pairs, rows and
columns: the coarse transform on the band-rotation kernels, and FP64 sums of few
rows on matrix-core tiles."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_split import run, test_coarse_transform_forms as coarse_round_trip  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nw,na,box,m", [
    (1, 17, 1, (8, 8, 2), (2, 2, 1)), (1, 17, 1, (8, 8, 1), (2, 2, 1)),     # 512 and 256 pairs
    (0, 17, 1, (8, 8, 4), (2, 2, 1)), (0, 17, 1, (8, 8, 2), (2, 2, 1)),     # 1024 and 512
    (1, 9, 5, (8, 8, 2), (2, 2, 1)), (0, 9, 5, (8, 8, 1), (2, 2, 1)),       # 15 modes
    (1, 12, 9, (8, 8, 2), (2, 2, 1)),                                       # 27 modes: rotations alone
])
def test_coarse_forms(run, prec, nw, na, box, m):  # noqa: F811
    coarse_round_trip(run, prec, nw, na, box, m)


@pytest.mark.parametrize("nq,ne", [(4, 436), (4, 437), (5, 437), (8, 873), (8, 874), (9, 874)])
def test_fp64_few_rows(run, nq, ne):  # noqa: F811
    """75 columns a lattice vector: around 32768 and 65536 columns."""
    rp = synth.box((5, 13, 1))
    s = synth.make_system(5, 1, synth.box((ne, 1, 1)), rp, [nq, 52])
    q = np.random.default_rng(nq).random((nq, 3))
    ph, g = oracle.phases(q, rp), s.g.reshape(65, -1)
    got = run.phase_sum_rp(run.system(s), q, 0).reshape(nq, -1)
    mag = np.abs(ph) @ (np.abs(g.real) + np.abs(g.imag))
    assert np.all(np.abs(got - ph @ g) <= 2 * (2 * 65 + 4) * 2.0 ** -53 * mag)
