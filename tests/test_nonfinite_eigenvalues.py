"""Points that are not finite: their eigensolves end with NaN eigenvalues, whose
order must stay a permutation (it indexes memory), raise EPHW_ENOCONV and leave
the other points of the call as they are."""
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_places_are_a_permutation(tmp_path):
    from paper_2603_10295_amd import build as b
    exe = str(tmp_path / "check")
    r = subprocess.run([b.hipcc(), f"--offload-arch={b.ARCH}", "--offload-host-only", "-x", "hip", "-std=c++17",
                        os.path.join(ROOT, "tests", "ascending_place_check.hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ascending_place_check: ok" in r.stdout, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("nw", [3, 11, 20, 36])
def test_bands_of_points_that_are_not_finite(nw):
    import torch
    from paper_2603_10295_amd import ephw
    ctx = ephw.Context(0)
    sysh = ephw.System.from_synth(ctx, synth.make_system(nw, 1, synth.box((3, 1, 1)), synth.box((1, 1, 1)), [nw, 8]))
    k = np.random.default_rng(nw).random((9, 3))

    def bands():
        eps = torch.empty((9, nw), dtype=torch.float64, device="cuda:0")
        vec = torch.empty((9, nw, nw), dtype=torch.complex128, device="cuda:0")
        ephw.bands(sysh, torch.from_numpy(k).to("cuda:0"), eps, vec)
        torch.cuda.synchronize()
        return eps.cpu().numpy(), vec.cpu().numpy()
    eps, vec = bands()
    ctx.check()
    k[2, 0], k[5, 1] = np.nan, np.inf
    got, gvec = bands()
    with pytest.raises(ephw.EphwError) as e:
        ctx.check()
    assert e.value.status == ephw.ENOCONV
    fine = np.isfinite(k).all(1)
    assert np.array_equal(got[fine], eps[fine]) and np.array_equal(gvec[fine], vec[fine])
    assert not np.isfinite(got[~fine]).any()
    sysh.close()
    ctx.close()
