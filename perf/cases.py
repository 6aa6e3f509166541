"""Performance cases of the electron-phonon interpolation: what programs call, through the public Python binding.

A case is one call (or the few calls that belong together) as a program makes it on prepared handles: a System with its g(Re,Rp) on the
device and a KSet of the fine k list.  Shapes are those of the bench workloads (Si-like, MoS2-like, nanoribbon, the
multi-system batch, the coarse transform, the energy window, the linewidth) at one chunk of their q lists, and of the tests' toys.

  interp    ephw.interpolate on a chunk of q points (k+q on the k grid, or off it with its own eigensolves)
  pairs     ephw.window_pairs, then ephw.interpolate_pairs on the kept pairs
  linewidth ephw.interpolate_linewidth (g reduced as it is formed)
  grad      autograd.eph_loss forward and backward (gradients of g, k and q), k-sets included as in a training step
  adjoint   ephw.loss_backward on a prepared k-set (wide systems)
  batch     ephw.Batch of several systems in one pass
  coarse    ephw.wannier_transform, coarse Bloch -> Wannier

Tensors follow the seeded generators of the bench: complex normal g damped by exp(-(|Re|+|Rp|)/2), Hermitian-paired H(R) and C(R)
damped by exp(-|R|), masses and (with "ws") Wigner-Seitz weights 1/n.
"""
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2603_10295_amd import ephw
from paper_2603_10295_amd.autograd import eph_loss

DEV = "cuda:0" if torch.cuda.is_available() else "cpu"
PRECS = {"fp64": ephw.FP64, "fp32": ephw.FP32, "comp": ephw.FP32_COMP}


def listed():
    return [
        # the README's toy: one small call, launches and latency
        dict(name="toy_fp64", op="interp", nw=8, na=2, re="5x5x5", rp="5x5x5", prec="fp64", k="16", nq=16, out="g", ws=False),
        # a training step on a small model system, k-sets created inside as autograd does
        dict(name="toy_grad_fp64", op="grad", nw=4, na=1, re="3x3x3", rp="3x3x3", prec="fp64", k="4x4x4", nq=8),
        # MoS2-like sheet, random in-plane points: k+q off the grid, an eigensolve per pair
        dict(name="mos2_fp32", op="interp", nw=11, na=3, re="18x18x1", rp="18x18x1", prec="fp32", k="1000", nq=128, out="g", ws=False),
        # the same sheet in double precision, as a reference run does it, with Wigner-Seitz weights
        dict(name="mos2_fp64", op="interp", nw=11, na=3, re="18x18x1", rp="18x18x1", prec="fp64", k="1000", nq=64, out="g", ws=True),
        # dense Si, one q batch of the headline bench: g stored for 8000 k
        dict(name="si_dense_fp32", op="interp", nw=8, na=2, re="10x10x10", rp="10x10x10", prec="fp32", k="20x20x20", nq=128, out="g", ws=False),
        # a 16-band system in compensated FP32, ragged q count, g and band sums
        dict(name="mid_comp", op="interp", nw=16, na=3, re="6x6x6", rp="6x6x6", prec="comp", k="12x12x12", nq=45, out="g+sums", ws=True),
        # energy-window pass of dense Si: the lowest tenth of the lowest band
        dict(name="si_window_fp32", op="pairs", nw=8, na=2, re="10x10x10", rp="10x10x10", prec="fp32", k="20x20x20", nq=8000, keep=0.1),
        # phonon-limited linewidth of Si bands over a q chunk, g never stored
        dict(name="si_linewidth_fp32", op="linewidth", nw=8, na=2, re="8x8x8", rp="8x8x8", prec="fp32", k="20x20x20", nq=64),
        # nanoribbon (200 bands, 150 modes): band rotations dominate
        dict(name="ribbon_fp32", op="interp", nw=200, na=50, re="1x11x1", rp="1x11x1", prec="fp32", k="1x8x1", nq=8, out="g", ws=False),
        # gradients on a nanoribbon, the widest training step
        dict(name="ribbon_adjoint_fp32", op="adjoint", nw=200, na=50, re="1x5x1", rp="1x5x1", prec="fp32", k="1x8x1", nq=4),
        # several systems of mixed shapes in one captured pass
        dict(name="batch_fp32", op="batch", prec="fp32",
             items="22,4,5x6x4,6;9,2,6x7x5,8;4,1,4x4x4,6;31,3,4x5x6,5;13,5,5x4x6,6;8,2,8x7x6,9;27,1,6x5x4,6;17,2,5x5x7,7"),
        # coarse Bloch -> Wannier transform of Si
        dict(name="coarse_si_fp32", op="coarse", nw=8, na=2, re="8x8x8", rp="4x4x4", prec="fp32"),
    ]


# --- shapes and costs ---------------------------------------------------------

def _dims(text):
    return [int(x) for x in text.split("x")]


def _count(text):
    return math.prod(_dims(text))


def _size(c):
    """nw, nm, ne, np, nk, nq of a case (not of a batch)."""
    ne, np_ = _count(c["re"]), _count(c["rp"])
    nk, nq = (ne, np_) if c["op"] == "coarse" else (_count(c["k"]), c["nq"])
    return c["nw"], 3 * c["na"], ne, np_, nk, nq


def _csize(c):
    return 16 if c["prec"] == "fp64" else 8


def _eig_flops(n):
    return 36.0 * n ** 3


def _interp_work(nw, nm, ne, np_, nk, nq, cs, off_grid, out_bytes):
    e = nm * nw * nw
    fl = 8.0 * nq * np_ * ne * e + 8.0 * nk * nq * ne * e + 16.0 * nk * nq * nm * nw ** 3 + 8.0 * nq * ne * nm * e
    fl += nq * (8.0 * np_ * nm * nm + _eig_flops(nm))
    by = np_ * ne * e * cs + out_bytes + nk * (ne * cs + nw * nw * cs) + nq * 24.0
    if off_grid:
        fl += nk * nq * (8.0 * ne * nw * nw + _eig_flops(nw))
    else:
        by += 4.0 * nk * nq
    return fl, by


def work(c):
    cs = _csize(c)
    if c["op"] == "batch":
        fl = by = 0.0
        for s in _batch_items(c):
            nw, nm, ne, np_, nk, nq = _size(s)
            f, b = _interp_work(nw, nm, ne, np_, nk, nq, cs, False, nk * nq * nm * 8.0)
            fl, by = fl + f, by + b
        return {"bytes": by, "flops": fl}
    nw, nm, ne, np_, nk, nq = _size(c)
    e = nm * nw * nw
    if c["op"] == "interp":
        off = "x" not in c["k"]
        out = nk * nq * (e * cs * ("g" in c["out"].split("+")) + 8.0 * nm * ("sums" in c["out"]) + 8.0 * nw * off) + nq * nm * 8.0
        fl, by = _interp_work(nw, nm, ne, np_, nk, nq, cs, off, out)
    elif c["op"] == "pairs":
        nka = max(1, round(c["keep"] * nk))
        kept = c["keep"] * nka * nq     # k+q inside the window for about the same share
        fl = 8.0 * min(nka, nq) * ne * np_ * e + 8.0 * kept * min(ne, np_) * e + 8.0 * kept * e * nm
        fl += nq * (8.0 * np_ * nm * nm + _eig_flops(nm))
        by = np_ * ne * e * cs + 4.0 * nk * nq + kept * (8.0 + nm * cs) + nk * (ne + nw) * cs
    elif c["op"] == "linewidth":
        fl, by = _interp_work(nw, nm, ne, np_, nk, nq, cs, False, nk * nw * 8.0)
    elif c["op"] in ("grad", "adjoint"):
        f, b = _interp_work(nw, nm, ne, np_, nk, nq, cs, False, 0.0)
        fl, by = 3.0 * f, 2.0 * b
        if c["op"] == "grad":
            fl += nk * _eig_flops(nw)
    else:
        fl = 8.0 * (2 * nk * nq * nm * nw ** 3 + ne * nq * e * nk + nq * ne * nm * e + np_ * ne * e * nq)
        by = (nk * nq * e + np_ * ne * e) * cs + 4.0 * nk * nq
    return {"bytes": by, "flops": fl}


def _cost(c):
    """work in FP32-flop terms (FP64 and the compensated form run slower), and the device bytes of a state."""
    f = work(c)["flops"] * {"fp64": 2.2, "comp": 1.2, "fp32": 1.0}[c["prec"]]
    if c["op"] == "batch":
        g = sum(8.0 * _size(s)[2] * _size(s)[3] * _size(s)[1] * s["nw"] ** 2 for s in _batch_items(c))
        return f, g + 24e9 * 0.1
    nw, nm, ne, np_, nk, nq = _size(c)
    g = _csize(c) * ne * np_ * nm * nw * nw
    out = 0.0 if c["op"] in ("pairs", "linewidth") else _csize(c) * nk * nq * nm * nw * nw
    return f, g + out


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every op and precision, sizes over the whole ranges (odd ones among them)."""
    big = _cost(listed()[4])
    while True:
        op = rng.choice(["interp"] * 6 + ["pairs", "linewidth", "grad", "adjoint", "batch", "coarse"])
        prec = rng.choice(["fp32", "fp32", "fp64", "comp"]) if op == "interp" else rng.choice(["fp32", "fp32", "fp64"])
        box = "x".join(str(rng.randint(3, 10)) for _ in range(3)) if rng.random() < 0.7 else "%dx%dx1" % (rng.randint(5, 18), rng.randint(5, 18))
        grid = "x".join(str(_log(rng, 4, 20)) for _ in range(3))
        c = dict(op=op, nw=_log(rng, 4, 32), na=rng.randint(1, 8), re=box, rp=box, prec=prec)
        if op == "interp":
            if rng.random() < 0.2:                                   # a ribbon
                box = "1x%dx1" % (2 * rng.randint(2, 5) + 1)
                c.update(nw=_log(rng, 33, 200), na=rng.randint(8, 50), re=box, rp=box, prec=rng.choice(["fp32", "fp64"]))
                c.update(k="1x%dx1" % rng.randint(4, 16), nq=rng.randint(2, 12), out=rng.choice(["g", "sums"]), ws=False)
            else:
                c.update(k=grid if rng.random() < 0.5 else str(_log(rng, 16, 2000)), nq=_log(rng, 1, 300),
                         out=rng.choice(["g", "g", "g+sums", "sums"]), ws=rng.random() < 0.4)
        elif op == "pairs":
            c.update(k=grid, nq=0, keep=round(rng.uniform(0.05, 0.4), 2), na=rng.randint(1, 3))
        elif op == "linewidth":
            c.update(k=grid, nq=_log(rng, 1, 200), prec=rng.choice(["fp32", "fp64"]))
        elif op == "grad":
            c.update(nw=_log(rng, 3, 16), na=rng.randint(1, 3), re="3x4x3", rp="3x3x4", k="x".join(str(rng.randint(2, 5)) for _ in range(3)), nq=rng.randint(2, 12))
        elif op == "adjoint":
            box = "1x%dx1" % (2 * rng.randint(1, 3) + 1)
            c.update(nw=_log(rng, 33, 200), na=rng.randint(8, 50), re=box, rp=box, prec="fp32", k="1x%dx1" % rng.randint(4, 10), nq=rng.randint(2, 6))
        elif op == "batch":
            items = ";".join("%d,%d,%s,%d" % (_log(rng, 4, 32), rng.randint(1, 6), "x".join(str(rng.randint(4, 8)) for _ in range(3)), rng.randint(4, 9))
                             for _ in range(rng.randint(2, 8)))
            c = dict(op=op, prec=rng.choice(["fp32", "fp32", "fp64"]), items=items)
        else:
            a = [rng.choice([4, 6, 8, 9]) for _ in range(3)]
            c.update(re="x".join(map(str, a)), rp="x".join(str(x if x < 6 else x // 2 if x % 2 == 0 else x // 3) for x in a))
        if "k" in c and "x" in c["k"]:
            n = _count(c["k"])
            c["nq"] = n if op == "pairs" else min(c["nq"], n)
        f, mem = _cost(c)
        if f <= big[0] and mem <= big[1] and (op != "adjoint" or mem < 4e9):
            return c


# --- inputs -------------------------------------------------------------------

def _box(text):
    """Integer lattice vectors -floor(n/2) .. ceil(n/2)-1 of each axis, lexicographic."""
    axes = [np.arange(-(n // 2), -(n // 2) + n) for n in _dims(text)]
    return np.stack([a.reshape(-1) for a in np.meshgrid(*axes, indexing="ij")], 1).astype(np.int32)


def _grid(text):
    axes = [np.arange(n) / n for n in _dims(text)]
    return np.stack([a.reshape(-1) for a in np.meshgrid(*axes, indexing="ij")], 1)


def _paired(r, n, rng, real):
    """M(R) with M(-R) = M(R)^dagger, damped by exp(-|R|); zero where -R is outside the box."""
    z = rng.standard_normal((len(r), n, n)) if real else (rng.standard_normal((len(r), n, n)) + 1j * rng.standard_normal((len(r), n, n))) / math.sqrt(2)
    at = {tuple(v): i for i, v in enumerate(r.tolist())}
    p = np.array([at.get(tuple(-x for x in v), -1) for v in r.tolist()])
    m = (z + np.conj(np.swapaxes(z[p], 1, 2))) / math.sqrt(2)
    m[p < 0] = 0
    return m * np.exp(-np.linalg.norm(r, axis=1))[:, None, None]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7fffffff)


def _system(c, seed):
    """Host tensors of a system and its g on the device."""
    rng = np.random.default_rng([seed, c["nw"], c["na"]])
    re, rp = _box(c["re"]), _box(c["rp"])
    nw, nm = c["nw"], 3 * c["na"]
    s = dict(nw=nw, na=c["na"], r_e=re, r_p=rp, r_h=re, r_c=rp, h_r=_paired(re, nw, rng, False), c_r=_paired(rp, nm, rng, True),
             mass=rng.uniform(0.5, 2.0, c["na"]))
    if c.get("ws"):
        for key, r in (("w_e", re), ("w_p", rp)):
            s[key] = 1.0 / rng.choice([1, 1, 1, 2, 3, 4, 6, 12], len(r))
    g = torch.randn((len(rp), len(re), nm, nw, nw), dtype=torch.complex128 if c["prec"] == "fp64" else torch.complex64, device=DEV, generator=_gen(seed))
    for r, shape in ((re, (1, -1, 1, 1, 1)), (rp, (-1, 1, 1, 1, 1))):
        g *= torch.from_numpy(np.exp(-0.5 * np.linalg.norm(r, axis=1))).to(DEV, g.real.dtype).reshape(shape)
    return s, g


def _points(c, seed):
    """k list, q list (a chunk of the grid, or random) and the k+q table (or None), host arrays."""
    rng = np.random.default_rng([seed, 77])
    if "k" in c and "x" not in c["k"]:
        k, q = rng.random((int(c["k"]), 3)), rng.random((c["nq"], 3))
        flat = np.array(_dims(c["re"])) == 1
        k[:, flat] = 0
        q[:, flat] = 0
        return k, q, None
    n = np.array(_dims(c["re"] if c["op"] == "coarse" else c["k"]))
    k = _grid("x".join(map(str, n)))
    if c["op"] == "coarse":
        q = _grid(c["rp"])
    else:
        q = k[(rng.integers(len(k)) + np.arange(c["nq"])) % len(k)]
    ik, iq = torch.from_numpy(np.rint(k * n).astype(np.int32)), torch.from_numpy(np.rint(q * n).astype(np.int32))
    t = torch.zeros((len(q), len(k)), dtype=torch.int32, device=DEV)
    for d in range(3):
        t = t * int(n[d]) + (ik[:, d].to(DEV)[None] + iq[:, d].to(DEV)[:, None]) % int(n[d])
    return k, q, t


def _window(e0, keep):
    """Window of the lowest share `keep` of one band's energies, its upper edge between two of them."""
    e = np.sort(e0)
    n = min(max(1, round(keep * len(e))), len(e) - 1)
    return float(e[0] - 1.0), float(0.5 * (e[n - 1] + e[n]))


def _lw_params(eps):
    span = float(eps.max() - eps.min())
    return dict(temperature=0.02 * span, mu=float(np.median(eps)), sigma=0.01 * span, omega_min=1e-3)


def _batch_items(c):
    out = []
    for t in c["items"].split(";"):
        nw, na, box, m = t.split(",")
        out.append(dict(op="interp", nw=int(nw), na=int(na), re=box, rp=box, prec=c["prec"], k="x".join([m] * 3), nq=int(m) ** 3, out="sums", ws=False))
    return out


def _bloch(c, seed):
    nw, nm, ne, np_, nk, nq = _size(c)
    return torch.randn((nq, nk, nm, nw, nw), dtype=torch.complex128 if c["prec"] == "fp64" else torch.complex64, device=DEV, generator=_gen(seed + 1))


def _to(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _load(ctx, c, seed):
    s, g = _system(c, seed)
    sysh = ephw.System(ctx, g=None, g_dtype=ephw.C128 if c["prec"] == "fp64" else ephw.C64, **s)
    sysh.set_g(g)
    return sysh, g


def prepare(case, seed):
    c = case
    ctx = ephw.Context(0)
    st = dict(case=c, ctx=ctx)
    if c["op"] == "batch":
        items, keep = [], []
        for i, s in enumerate(_batch_items(c)):
            sysh, _ = _load(ctx, s, seed + 1000 * i)
            k, q, t = _points(s, seed + 1000 * i)
            ks = ephw.KSet(sysh, _to(k), PRECS[s["prec"]])
            items.append(dict(ks=ks, q=_to(q), kq_index=t, flags=ephw.OUT_BAND_SUM | ephw.OUT_LOSS, loss_seed=7 + i,
                              band_sum=torch.empty((len(q), len(k), sysh.nm), dtype=torch.float64, device=DEV),
                              loss=torch.zeros(1, dtype=torch.float64, device=DEV)))
            keep.append(sysh)
        torch.cuda.synchronize()
        st.update(items=items, keep=keep, batch=ephw.Batch(ctx, items))
        return st
    sysh, g = _load(ctx, c, seed)
    k, q, t = _points(c, seed)
    st.update(sys=sysh, k=_to(k), q=_to(q), kqi=t)
    nk, nq, nm, nw = len(k), len(q), sysh.nm, sysh.nw
    prec = PRECS[c["prec"]]
    if c["op"] == "grad":
        st["leaves"] = (g.requires_grad_(True), st["k"].requires_grad_(True), st["q"].requires_grad_(True))
        return st
    st["ks"] = ks = ephw.KSet(sysh, st["k"], prec)
    f64 = dict(dtype=torch.float64, device=DEV)
    if c["op"] == "interp":
        want = c["out"].split("+")
        st["flags"] = (ephw.OUT_G if "g" in want else 0) | (ephw.OUT_BAND_SUM if "sums" in want else 0)
        o = {"omega": torch.empty((nq, nm), **f64)}
        if "g" in want:
            o["g_out"] = torch.empty((nq, nk, nm, nw, nw), dtype=g.dtype, device=DEV)
        if "sums" in want:
            o["band_sum"] = torch.empty((nq, nk, nm), **f64)
        if t is None:
            o["eps_kq"] = torch.empty((nq, nk, nw), **f64)
        st["o"] = o
    elif c["op"] in ("pairs", "linewidth"):
        eps = torch.empty((nk, nw), **f64)
        ks.bands(eps)
        eps = eps.cpu().numpy()
        if c["op"] == "pairs":
            st["window"] = _window(eps[:, 0], c["keep"])
        else:
            st["gamma"], st["lw"] = torch.empty((nk, nw), **f64), _lw_params(eps)
    elif c["op"] == "adjoint":
        st["o"] = dict(loss=torch.empty(1, **f64), dL_dg=torch.empty_like(g), dL_dk=torch.empty((nk, 3), **f64), dL_dq=torch.empty((nq, 3), **f64))
    else:
        st["bloch"], st["out"] = _bloch(c, seed), torch.empty_like(g)
    return st


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "interp":
        ephw.interpolate(state["ks"], state["q"], kq_index=state["kqi"], flags=state["flags"], **state["o"])
        return state["o"]
    if op == "pairs":
        lo, hi = state["window"]
        order, start, other, kq, bands = ephw.window_pairs(state["ks"], state["kqi"], lo, hi)
        n, nb = int(start[-1]), bands[1]
        g = torch.empty((n, state["sys"].nm, nb, nb), dtype=torch.complex128 if c["prec"] == "fp64" else torch.complex64, device=DEV)
        ephw.interpolate_pairs(state["ks"], state["q"], order, start, other, kq, bands=bands, g_out=g)
        return dict(start=start, other=other[:n], kq=kq[:n], g=g)
    if op == "linewidth":
        state["gamma"].zero_()
        ephw.interpolate_linewidth(state["ks"], state["q"], state["gamma"], kq_index=state["kqi"], **state["lw"])
        return state["gamma"]
    if op == "grad":
        for x in state["leaves"]:
            x.grad = None
        g, k, q = state["leaves"]
        loss = eph_loss(state["sys"], g, k, q, state["kqi"], 3)
        loss.backward()
        return dict(loss=loss.detach(), dg=g.grad, dk=k.grad, dq=q.grad)
    if op == "adjoint":
        for x in state["o"].values():
            x.zero_()
        ephw.loss_backward(state["ks"], state["q"], state["kqi"], loss_seed=3, **state["o"])
        return state["o"]
    if op == "batch":
        for it in state["items"]:
            it["loss"].zero_()
        state["batch"].run()
        return [(it["band_sum"], it["loss"]) for it in state["items"]]
    ephw.wannier_transform(state["ks"], state["q"], state["kqi"], state["bloch"], state["out"])
    return state["out"]


# --- the same in 64 bits, plain torch and numpy --------------------------------

C128 = torch.complex128


def _phase(p, r, w=None):
    t = p @ _to(r).to(p.dtype).T
    t = 2 * math.pi * (t - torch.round(t.detach()))
    ph = torch.complex(torch.cos(t), torch.sin(t))
    return ph if w is None else ph * _to(w)


def _eigh(h):
    """Ascending eigenvalues and column eigenvectors, the largest entry of each real and positive; LAPACK on several threads."""
    a = h.detach().cpu().numpy().reshape(-1, h.shape[-1], h.shape[-1])
    parts = np.array_split(a, min(len(a), 256))
    with ThreadPoolExecutor(16) as ex:
        got = list(ex.map(np.linalg.eigh, parts))
    e, v = np.concatenate([x[0] for x in got]), np.concatenate([x[1] for x in got])
    top = np.take_along_axis(v, np.abs(v).argmax(1)[:, None, :], 1)
    v = v * (np.conj(top) / np.abs(top))
    return _to(e.reshape(h.shape[:-1])), _to(v.reshape(h.shape))


def _hk(s, k, w=True):
    return torch.tensordot(_phase(k, s["r_h"]), _to(s["h_r"]), 1)


def _dq(s, q):
    m = np.repeat(s["mass"], 3)
    return torch.tensordot(_phase(q, s["r_c"]), _to(s["c_r"] / np.sqrt(m[:, None] * m[None])).to(C128), 1)


def _modes(s, q):
    lam, e = _eigh(_dq(s, q))
    return lam.abs().sqrt(), e / _to(np.sqrt(np.repeat(s["mass"], 3)))[None, :, None]


def _g_re_q(s, g, q):
    """Eq. (9) for a few q: [q][Re][ka][m'n']."""
    ph, flat = _phase(q, s["r_p"], s.get("w_p")), g.reshape(g.shape[0], -1)
    out = torch.empty((len(q), flat.shape[1]), dtype=C128, device=DEV)
    step = max(1, int(4e8 // flat.shape[0]))
    for a in range(0, flat.shape[1], step):
        out[:, a:a + step] = ph @ flat[:, a:a + step].to(C128)
    return out.reshape(len(q), g.shape[1], g.shape[2], -1)


def _g_bloch(s, g, k, q, vk, vkq_of, u):
    """g(k,q) of Eq. (7), one q after the other: yields [k][nu][m][n]."""
    pk, nw = _phase(k, s["r_e"], s.get("w_e")), s["nw"]
    for a in range(0, len(q), 16):
        gq = _g_re_q(s, g, q[a:a + 16])
        for i in range(gq.shape[0]):
            x = torch.matmul(u[a + i].T.contiguous(), gq[i])                                # [Re][nu][m'n']
            w = (pk @ x.reshape(len(x), -1)).reshape(len(k), -1, nw, nw)
            yield torch.matmul(torch.matmul(vkq_of(a + i).conj().transpose(1, 2).contiguous()[:, None], w), vk[:, None])


def _exact_interp(c, seed):
    s, g = _system(c, seed)
    k, q, t = _points(c, seed)
    k, q = _to(k), _to(q)
    om, u = _modes(s, q)
    ek, vk = _eigh(_hk(s, k))
    if t is None:
        ekq, vkq = _eigh(_hk(s, (q[:, None] + k[None]).reshape(-1, 3)).reshape(len(q), len(k), s["nw"], s["nw"]))
        of = lambda i: vkq[i]                                                               # noqa: E731
    else:
        of = lambda i: vk[t[i].long()]                                                      # noqa: E731
    return s, k, q, t, om, u, ek, vk, of, (ekq if t is None else None), _g_bloch(s, g, k, q, vk, of, u)


def _weights(seed, index):
    """0.5 + the top 24 bits of the index-th SplitMix64 output."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (index.astype(np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return 0.5 + (z >> np.uint64(40)).astype(np.float64) * 2.0 ** -24


def _exact_grad(c, seed):
    s, g = _system(c, seed)
    k, q, t = _points(c, seed)
    k, q, g = _to(k).requires_grad_(True), _to(q).requires_grad_(True), g.to(C128).requires_grad_(True)
    nk, nq, nw, nm = len(k), len(q), s["nw"], 3 * s["na"]
    hk, dq = _hk(s, k).cpu(), _dq(s, q).cpu()
    hkq = _hk(s, (q[:, None] + k[None]).reshape(-1, 3)).cpu()
    vk, vkq = torch.linalg.eigh(hk)[1].to(DEV), torch.linalg.eigh(hkq)[1].to(DEV).reshape(nq, nk, nw, nw)
    u = torch.linalg.eigh(dq)[1].to(DEV) / _to(np.sqrt(np.repeat(s["mass"], 3)))[None, :, None]
    pq, pk = _phase(q, s["r_p"]), _phase(k, s["r_e"])
    loss = 0.0
    gq = (pq @ g.reshape(len(g), -1)).reshape(nq, g.shape[1], nm, -1)
    for i in range(nq):
        x = torch.matmul(u[i].T.contiguous(), gq[i])
        w = (pk @ x.reshape(len(x), -1)).reshape(nk, nm, nw, nw)
        y = torch.matmul(torch.matmul(vkq[i].conj().transpose(1, 2).contiguous()[:, None], w), vk[:, None])
        n = nk * nm * nw * nw
        wt = _to(_weights(3, np.arange(i * n, (i + 1) * n))).reshape(y.shape)
        loss = loss + (wt * (y.real ** 2 + y.imag ** 2)).sum()
    dg, dk, dqq = torch.autograd.grad(loss, (g, k, q))
    return loss.detach(), dg, dk, dqq


def _exact_pairs(c, seed):
    s, g = _system(c, seed)
    k, q, t = _points(c, seed)
    k, q = _to(k), _to(q)
    ek, vk = _eigh(_hk(s, k))
    lo, hi = _window(ek[:, 0].cpu().numpy(), c["keep"])
    inside = (ek >= lo) & (ek <= hi)
    bands = inside.any(0).nonzero().reshape(-1)
    b0, nb = int(bands[0]), int(bands[-1] - bands[0]) + 1
    act = inside.any(1)
    keep = act[t.long()] & act[None]                                                         # [q][k]
    by_k = int(keep.any(0).sum()) < int(keep.any(1).sum())
    own = keep.T if by_k else keep
    n = own.sum(1)
    om, u = _modes(s, q)
    first, second = (_phase(k, s["r_e"]), _phase(q, s["r_p"])) if by_k else (_phase(q, s["r_p"]), _phase(k, s["r_e"]))
    src = (g.transpose(0, 1) if by_k else g).reshape(g.shape[1] if by_k else g.shape[0], -1)
    out, nw, nm = [], s["nw"], 3 * s["na"]
    rows = n.nonzero().reshape(-1)
    inner = g.shape[0] if by_k else g.shape[1]
    vkb = vk[:, :, b0:b0 + nb]
    per = max(1, int(2e9 // (16 * src.shape[1])))
    for a in range(0, len(rows), per):
        r = rows[a:a + per]
        g1 = torch.empty((len(r), src.shape[1]), dtype=C128, device=DEV)
        step = max(1, int(1e8 // src.shape[0]))
        for b in range(0, src.shape[1], step):
            g1[:, b:b + step] = first[r] @ src[:, b:b + step].to(C128)
        for i, j in enumerate(r.tolist()):
            o = own[j].nonzero().reshape(-1)
            w = (second[o] @ g1[i].reshape(inner, -1)).reshape(len(o), nm, -1)
            qq, kk = (o, torch.full_like(o, j)) if by_k else (torch.full_like(o, j), o)
            w = torch.matmul(u[qq].transpose(1, 2).contiguous(), w).reshape(len(o), nm, nw, nw)
            vq = vkb[t[qq, kk].long()].conj().transpose(1, 2).contiguous()
            out.append(torch.matmul(torch.matmul(vq[:, None], w), vkb[kk][:, None]))
    return dict(start=None, other=None, kq=None, g=torch.cat(out))


def _exact_linewidth(c, seed):
    s, k, q, t, om, u, ek, vk, of, _, gs = _exact_interp(c, seed)
    p = _lw_params(ek.cpu().numpy())
    tt, sg = p["temperature"], p["sigma"]
    gamma = torch.zeros_like(ek)
    gauss = lambda x: torch.exp(-0.5 * (x / sg) ** 2) / (sg * math.sqrt(2 * math.pi))        # noqa: E731
    for i, g in enumerate(gs):
        g2 = g.real ** 2 + g.imag ** 2                                                       # [k][nu][m][n]
        o = om[i]
        use = (o >= p["omega_min"]) & (o > 0)
        nb = torch.where(use, 1 / torch.expm1(torch.where(use, o, torch.ones_like(o)) / tt), torch.zeros_like(o))
        amp = torch.where(use, 0.5 / torch.where(use, o, torch.ones_like(o)), torch.zeros_like(o))
        em = ek[t[i].long()]
        fm = torch.sigmoid(-(em - p["mu"]) / tt)[:, None, :, None]
        de = (ek[:, None, :] - em[:, :, None])[:, None]                                      # [k][1][m][n]
        n_, o_, a_ = nb[None, :, None, None], o[None, :, None, None], amp[None, :, None, None]
        gamma += (a_ * ((n_ + fm) * gauss(de + o_) + (n_ + 1 - fm) * gauss(de - o_)) * g2).sum((1, 2))
    return math.pi / len(q) * gamma


def _exact_coarse(c, seed):
    s, _ = _system(c, seed)
    k, q, t = _points(c, seed)
    k, q = _to(k), _to(q)
    _, vk = _eigh(_hk(s, k))
    _, u = _modes(s, q)
    b = _bloch(c, seed)
    pe, pp = _phase(k, s["r_e"]).conj(), _phase(q, s["r_p"]).conj()
    mid = []
    for i in range(len(q)):
        x = torch.matmul(torch.matmul(vk[t[i].long()][:, None], b[i].to(C128)), vk.conj().transpose(1, 2).contiguous()[:, None])
        x = torch.matmul(torch.linalg.inv(u[i].cpu()).to(DEV).T.contiguous(), x.reshape(len(k), u.shape[1], -1))
        mid.append(pe.T.contiguous() @ x.reshape(len(k), -1))
    out = pp.T.contiguous() @ torch.stack(mid).reshape(len(q), -1)
    return (out / (len(k) * len(q))).reshape(len(q), len(k), u.shape[1], s["nw"], s["nw"])


def exact(case, seed):
    """run()'s outputs in 64 bits; None where the plain form would take too long."""
    c = case
    op = c["op"]
    if op == "batch":
        out = []
        for i, s in enumerate(_batch_items(c)):
            sums, loss = [], 0.0
            for j, g in enumerate(_exact_interp(s, seed + 1000 * i)[-1]):
                g2 = g.real ** 2 + g.imag ** 2
                sums.append(g2.sum((2, 3)))
                loss += float((_to(_weights(7 + i, np.arange(j * g2.numel(), (j + 1) * g2.numel()))).reshape(g2.shape) * g2).sum())
            out.append((torch.stack(sums), torch.tensor([loss], dtype=torch.float64)))
        return out
    if op == "pairs":
        return _exact_pairs(c, seed)
    if op == "linewidth":
        return _exact_linewidth(c, seed)
    if op == "coarse":
        return _exact_coarse(c, seed)
    if op in ("grad", "adjoint"):
        loss, dg, dk, dq = _exact_grad(c, seed)
        return dict(loss=loss, dg=dg, dk=dk, dq=dq) if op == "grad" else dict(loss=loss.reshape(1), dL_dg=dg, dL_dk=dk, dL_dq=dq)
    s, k, q, t, om, u, ek, vk, of, ekq, gs = _exact_interp(c, seed)
    want = c["out"].split("+")
    o = {"omega": om}
    g_out = torch.empty((len(q), len(k), 3 * s["na"], s["nw"], s["nw"]), dtype=C128, device=DEV) if "g" in want else None
    sums = []
    for i, g in enumerate(gs):
        if g_out is not None:
            g_out[i] = g
        if "sums" in want:
            sums.append((g.real ** 2 + g.imag ** 2).sum((2, 3)))
    if g_out is not None:
        o["g_out"] = g_out
    if sums:
        o["band_sum"] = torch.stack(sums)
    if t is None:
        o["eps_kq"] = ekq
    return o
