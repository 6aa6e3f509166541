"""The sweep limit of the eigensolves above order 32: around the number of
launches that run one sweep each, and at the largest limit; too small a limit is
reported."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [33, 70])
def test_limits_give_the_same_bands(nw):
    import torch
    from paper_2603_10295_amd import ephw
    ctx = ephw.Context(0)
    sysh = ephw.System.from_synth(ctx, synth.make_system(nw, 1, synth.box((3, 1, 1)), synth.box((1, 1, 1)), [nw, 9]))
    k = torch.from_numpy(np.random.default_rng(1).random((3, 3))).to("cuda:0")

    def bands(limit):
        ctx.set_limits(max_sweeps=limit)
        eps = torch.empty((3, nw), dtype=torch.float64, device="cuda:0")
        vec = torch.empty((3, nw, nw), dtype=torch.complex128, device="cuda:0")
        ephw.bands(sysh, k, eps, vec)
        return eps, vec
    ref = bands(40)
    ctx.check()
    for limit in (15, 16, 17, 18, 1000):
        got = bands(limit)
        ctx.check()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    for limit in (0, 1, 3):
        bands(limit)
        with pytest.raises(ephw.EphwError) as e:
            ctx.check()
        assert e.value.status == ephw.ENOCONV
    sysh.close()
    ctx.close()
