"""The FP32 phase sums on the 16-bit matrix cores (calls that return complex64
values alone): the BF16 form that splits as it loads and the packed FP16 form,
at the edges of their tiles, slabs and dispatch, against NumPy in 64 bits.

Bound of an element, from the format alone: every rounding of the running sum
is at most 2^-24 of sum |a b| (three accumulations per 16 terms in the packed
form, six in the BF16 form, and two roundings of the inputs to complex64), and
the parts a split leaves out are at most 2^-21 of it; a complex product has two
real ones per part."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def bound(K, steps):
    return 2 * ((steps * ((K + 15) // 16) + 4) * 2.0 ** -24 + 2.0 ** -21)


@pytest.fixture(scope="module")
def run():
    from gpu_run import Runner
    return Runner()


def system(box, nw, na, seed, ws=False, rp=((0, 0, 0),)):
    s = synth.make_system(nw, na, synth.box(box), np.asarray(rp, dtype=np.int32), [seed, 31], g_dtype=np.complex64)
    if ws:
        s = dataclasses.replace(s, w_e=1.0 / np.random.default_rng(seed).choice([1, 2, 3, 12], len(s.r_e)))
    return s


def re_sums(s, k):
    """sum_Re w e^{ik.Re} g(Re) in 64 bits and the sum of the terms' magnitudes, [k][ka][m'][n']"""
    ph, g = oracle.phases(k, s.r_e, s.w_e), s.g[0].reshape(len(s.r_e), -1).astype(np.complex128)
    shape = (len(k),) + s.g.shape[2:]
    return (ph @ g).reshape(shape), (np.abs(ph) @ (np.abs(g.real) + np.abs(g.imag))).reshape(shape)


def wannier(run, s, k, q, prec):
    from paper_2603_10295_amd import ephw
    return run.interpolate(run.system(s), k, q, prec, flags=ephw.OUT_G | ephw.OUT_WANNIER, want_eps_kq=False)["g"]


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("nk,box,nw,na,ws", [
    (40, (4, 4, 4), 5, 1, False),      # K = 64, the first that is split; 64-row tile
    (130, (5, 13, 1), 6, 2, True),     # K = 65, weights; two row tiles, the last of two rows
    (511, (5, 4, 4), 3, 1, False),     # K = 80, below the packed sets
    (512, (4, 4, 4), 5, 1, False),     # the first packed set
    (515, (5, 13, 1), 7, 2, True),     # packed: K, rows and columns ragged
    (640, (7, 6, 5), 8, 2, False),     # packed: whole tiles
])
def test_re_sum(run, prec, nk, box, nw, na, ws):
    s = system(box, nw, na, 3, ws)
    rng = np.random.default_rng(nk)
    k, q = rng.random((nk, 3)), np.array([[0.1, 0.2, 0.3], [0.7, 0.0, 0.4]])
    ref, mag = re_sums(s, k)
    got = wannier(run, s, k, q, prec)
    for j in range(len(q)):
        assert np.all(np.abs(got[j] - ref) <= bound(len(s.r_e), 6) * mag)


def test_packed_columns_of_any_scale(run):
    """Columns between 2^-100 and 2^100 keep their own relative accuracy; zero
    columns are zero, and a column that holds an infinity or a NaN is the only
    one that is not finite."""
    s = system((5, 13, 1), 6, 2, 5)
    g = s.g.copy()
    rng = np.random.default_rng(9)
    g *= (2.0 ** rng.integers(-100, 100, g.shape[2:])).astype(np.float32)
    g[0, :, 1, 2, 3] = 0
    g[0, 7, 2, 0, 1] = np.inf
    g[0, 9, 3, 4, 4] = np.nan
    s = dataclasses.replace(s, g=g)
    k, q = rng.random((600, 3)), np.zeros((1, 3))
    got = wannier(run, s, k, q, 1)[0]
    fine = np.ones(g.shape[2:], dtype=bool)
    fine[2, 0, 1] = fine[3, 4, 4] = False
    clean = dataclasses.replace(s, g=np.where(np.isfinite(g), g, 0).astype(np.complex64))
    ref, mag = re_sums(clean, k)
    assert np.all(np.abs(got - ref)[:, fine] <= bound(65, 6) * mag[:, fine])
    assert not np.any(got[:, 1, 2, 3])
    assert not np.any(np.isfinite(got[:, ~fine]))


def test_weights_beyond_the_packed_range(run):
    """Weights spread over more than 2^8 keep the set unpacked."""
    s = system((5, 13, 1), 4, 1, 6)
    w = np.ones(65)
    w[::2] = 1e-4
    s = dataclasses.replace(s, w_e=w, g=(s.g / w[None, :, None, None, None]).astype(np.complex64))
    k, q = np.random.default_rng(1).random((530, 3)), np.zeros((1, 3))
    ref, mag = re_sums(s, k)
    assert np.all(np.abs(wannier(run, s, k, q, 1)[0] - ref) <= bound(65, 6) * mag)


@pytest.mark.parametrize("nq", [17, 64, 65, 130])
@pytest.mark.parametrize("prec", [1, 2])
def test_rp_sum(run, prec, nq):
    rp = synth.box((5, 13, 1))
    s = system((2, 1, 1), 5, 1, 8, rp=rp)
    q = np.random.default_rng(nq).random((nq, 3))
    ph, g = oracle.phases(q, rp), s.g.reshape(65, -1).astype(np.complex128)
    ref, mag = ph @ g, np.abs(ph) @ (np.abs(g.real) + np.abs(g.imag))
    got = run.phase_sum_rp(run.system(s), q, prec).reshape(nq, -1)
    assert np.all(np.abs(got - ref) <= bound(65, 6) * mag)


@pytest.mark.parametrize("nk", [70, 520])
@pytest.mark.parametrize("nw,na", [(8, 2), (8, 1), (4, 1), (12, 1)])
def test_rotated_g_agrees_with_the_fp32_instructions(run, nk, nw, na):
    """g alone (split, packed from 512 points on) against g of a call that also
    returns the loss (FP32 instructions), in every fused rotation form: each
    within 1e-5 of the largest element of the other."""
    from paper_2603_10295_amd import ephw
    s = system((4, 4, 4), nw, na, 11, rp=synth.box((4, 4, 4)))
    rng = np.random.default_rng(2)
    k, q = rng.random((nk, 3)), rng.random((5, 3))
    h = run.system(s)
    a = run.interpolate(h, k, q, 1, flags=ephw.OUT_G, want_eps_kq=False)["g"]
    b = run.interpolate(h, k, q, 1, flags=ephw.OUT_G | ephw.OUT_LOSS, want_eps_kq=False)["g"]
    assert np.abs(a - b).max() <= 1e-5 * np.abs(b).max()


@pytest.mark.parametrize("nq,box", [(1, (1, 1, 1)), (4, (4, 4, 1)), (15, (17, 1, 1)), (16, (5, 13, 1)), (17, (5, 13, 1))])
def test_rp_sum_fp64_few_rows(run, nq, box):
    """FP64 sums of up to 16 q over at least 16384 columns take a 16-row tile:
    K below, at and past a slab, a ragged last column tile, and one row more."""
    rp = synth.box(box)
    s = synth.make_system(5, 1, synth.box((20, 11, 1)), rp, [nq, 32])
    q = np.random.default_rng(nq).random((nq, 3))
    K = len(rp)
    ph, g = oracle.phases(q, rp), s.g.reshape(K, -1)
    got = run.phase_sum_rp(run.system(s), q, 0).reshape(nq, -1)
    mag = np.abs(ph) @ (np.abs(g.real) + np.abs(g.imag))
    assert np.all(np.abs(got - ph @ g) <= 2 * (2 * K + 4) * 2.0 ** -53 * mag)


@pytest.mark.parametrize("prec,nw,na,box,m", [(1, 8, 2, (4, 4, 4), (2, 2, 2)), (0, 5, 1, (3, 2, 1), (3, 1, 1)),
                                              (1, 12, 9, (3, 3, 1), (3, 3, 1)), (1, 33, 1, (2, 2, 1), (2, 1, 1))])
def test_coarse_transform_forms(run, prec, nw, na, box, m):
    """Eq. (6) inverts Eq. (7) in each of its forms: rotations and modes on the
    small kernels, more than 24 modes, more than 32 bands."""
    import torch
    from paper_2603_10295_amd import ephw
    from gpu_run import cplx_dtype, dev
    s = synth.make_system(nw, na, synth.box(box), synth.box(m), [nw, 33],
                          g_dtype=np.complex128 if prec == 0 else np.complex64)
    k, q = synth.uniform_grid(box), synth.uniform_grid(m)
    n = np.asarray(box)
    ik, iq = np.rint(k * n).astype(int), np.rint(q * n).astype(int)
    t = (ik[None] + iq[:, None]) % n
    kqi = dev((t[..., 0] * n[1] * n[2] + t[..., 1] * n[2] + t[..., 2]).astype(np.int32))
    h = run.system(s)
    ks = ephw.KSet(h, dev(k), prec)
    gb = torch.empty((len(q), len(k), s.nm, nw, nw), dtype=cplx_dtype(prec), device="cuda:0")
    out = torch.empty(s.g.shape, dtype=cplx_dtype(prec), device="cuda:0")
    ephw.interpolate(ks, dev(q), kq_index=kqi, flags=ephw.OUT_G, g_out=gb)
    ephw.wannier_transform(ks, dev(q), kqi, gb, out)
    run.ctx.check()
    ks.close()
    # two passes of sums and unitary rotations over at most 64 terms each way
    assert np.abs(out.cpu().numpy() - s.g).max() <= (1e-12 if prec == 0 else 1e-5) * np.abs(s.g).max()


@pytest.mark.parametrize("order,nk,nq,fill,nw,na,tight", [
    ("by_k", 560, 700, 0.95, 3, 1, False),    # both sums packed; 27 columns a group, ragged last rows
    ("by_k", 560, 40, 0.9, 4, 1, False),      # the Re sum alone (few pairs per k)
    ("by_k", 560, 40, 0.9, 4, 1, True),       # the same without the memory for its operands
    ("by_q", 700, 5, 0.95, 3, 1, False),      # 135 columns in a batch, their last tile partly the next plane's
    ("by_q", 1100, 3, 0.55, 4, 2, False),     # several row and column tiles a group
])
def test_pairs_packed(run, order, nk, nq, fill, nw, na, tight):
    """Pair lists whose sums take packed operands, groups of different sizes and
    empty ones, Wannier gauge, against 64 bits: both sums' bounds."""
    import torch
    from paper_2603_10295_amd import ephw
    rng = np.random.default_rng(nk + nq)
    s = system((4, 17, 1), nw, na, 5, ws=True, rp=synth.box((13, 5, 1)))
    s = dataclasses.replace(s, w_p=1.0 / rng.choice([1, 2, 4], len(s.r_p)))
    k, q = rng.random((nk, 3)), rng.random((nq, 3))
    by_k = order == "by_k"
    keep = rng.random((nk, nq) if by_k else (nq, nk)) < fill
    if by_k:
        keep[3] = keep[17] = False
    start = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
    other = np.nonzero(keep)[1].astype(np.int32)
    h = run.system(s)
    ks = ephw.KSet(h, torch.from_numpy(k).cuda(), 1)
    args = (torch.from_numpy(q).cuda(), ephw.PAIRS_BY_K if by_k else ephw.PAIRS_BY_Q, start,
            torch.from_numpy(other).cuda(), torch.zeros(len(other), dtype=torch.int32, device="cuda"))
    g = torch.empty((len(other), s.nm, nw, nw), dtype=torch.complex64, device="cuda")

    def call():
        ephw.interpolate_pairs(ks, *args, flags=ephw.OUT_G | ephw.OUT_WANNIER, g_out=g)
        run.ctx.check()
    call()
    if tight:
        used = run.ctx.memory()[0]
        h.trim()
        g.zero_()
        run.ctx.set_limits(max_device_bytes=used - 4096)
        try:
            call()
        finally:
            run.ctx.set_limits()
        assert run.ctx.memory()[0] < used - 4096
    # 64 bits, [k][q][E] of the kept pairs
    pe, pp = (torch.from_numpy(x).cuda() for x in (oracle.phases(k, s.r_e, s.w_e), oracle.phases(q, s.r_p, s.w_p)))
    w = torch.from_numpy(s.g.astype(np.complex128)).cuda().reshape(len(s.r_p), len(s.r_e), -1)
    E = w.shape[2]

    def both(pe, w, pp):
        a = torch.mm(pe, w.permute(1, 0, 2).reshape(len(s.r_e), -1)).reshape(nk, len(s.r_p), E)
        return torch.mm(pp, a.permute(1, 0, 2).reshape(len(s.r_p), -1)).reshape(nq, nk, E)
    mag = both(pe.abs(), w.real.abs() + w.imag.abs(), pp.abs())
    ref = both(pe, w, pp)
    major = np.nonzero(keep)[0]
    ki, qi = (torch.from_numpy(x.astype(np.int64)).cuda() for x in ((major, other) if by_k else (other, major)))
    tol = 1.01 * (bound(len(s.r_e), 6) + bound(len(s.r_p), 6))
    assert bool(((g.reshape(-1, E) - ref[qi, ki]).abs() <= tol * mag[qi, ki]).all())
    ks.close()


@pytest.mark.parametrize("nk,nw,na", [(1, 3, 1), (64, 5, 1), (65, 3, 1), (130, 4, 2), (192, 3, 1)])
def test_compensated_rows(run, nk, nw, na):
    """The compensated FP32 sums of a call that also returns band sums, with
    64-row tiles (an odd number of them) and without: blocks of 32 k of two
    roundings each, then one per block."""
    from paper_2603_10295_amd import ephw
    s = system((5, 13, 1), nw, na, 9)
    k = np.random.default_rng(nk).random((nk, 3))
    got = run.interpolate(run.system(s), k, np.zeros((1, 3)), 2, want_eps_kq=False,
                          flags=ephw.OUT_G | ephw.OUT_BAND_SUM | ephw.OUT_WANNIER)["g"][0]
    ref, mag = re_sums(s, k)
    assert np.all(np.abs(got - ref) <= 2 * (64 + 65 // 32 + 4) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("nk", [40, 520])
def test_error_where_the_phases_agree(run, nk):
    """Both phase sums at q = 0 and around k = 0, where a one-sided rounding of
    the first sum would add up over the lattice vectors of the second: the
    error against 64 bits is no larger than that of the FP32 instructions (a
    call that also returns band sums)."""
    from paper_2603_10295_amd import ephw
    s = system((10, 10, 10), 8, 1, 13, rp=synth.box((8, 8, 8)))
    k = 1e-3 * np.random.default_rng(nk).random((nk, 3))
    q = np.zeros((1, 3))
    pe = oracle.phases(k, s.r_e)
    ref = (pe @ s.g.astype(np.complex128).sum(0).reshape(len(s.r_e), -1)).reshape(nk, s.nm, 8, 8)
    h = run.system(s)
    err = []
    for flags in (ephw.OUT_G, ephw.OUT_G | ephw.OUT_BAND_SUM):
        g = run.interpolate(h, k, q, 1, flags=flags | ephw.OUT_WANNIER, want_eps_kq=False)["g"][0]
        err.append(np.linalg.norm(g - ref) / np.linalg.norm(ref))
    assert err[0] <= err[1]
