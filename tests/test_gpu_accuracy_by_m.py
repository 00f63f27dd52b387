"""The FP32 pair path's rounding errors, m by m.

max|zeta| is set by the low m, so an error bound in it says little about a_lm at
m = 10.  Here each a_mm (one sum, S_{m,0}) and the gradient of zeta^10_{10,10} are
held to what plain FP32 arithmetic gives: the same steps in NumPy, one rounding
each, with (x - i y)^m by successive complex products and 64 partial sums.  All
pairs lie in the one shell, so no pair can change it by rounding."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1709_00086_amd import api

pytestmark = pytest.mark.gpu

F = np.float32
LMAX = 10
SLACK = 1.25  # of rms errors, over some hundred galaxies or more


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def ball(n, seed):
    """n galaxies in a ball of radius 50 about (100, 100, 100), float32."""
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(n, 3))
    v *= (50.0 * rng.uniform(size=(n, 1)) ** (1 / 3)) / np.linalg.norm(v, axis=1)[:, None]
    return (100.0 + v).astype(F), rng.uniform(0.5, 1.5, size=n)


def config(precision, basis="spin"):
    return api.Config(box=(110.0,) * 3, box_lo=(45.0,) * 3, rmax=101.0, nbins=1, lmax=LMAX,
                      periodic=False, precision=precision, basis=basis)


def fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(F)


def directions(d):
    """x and y of the FP32 unit vectors of FP32 separations [..., 3]."""
    x, y, z = d[..., 0], d[..., 1], d[..., 2]
    r2 = fma(z, z, fma(y, y, x * x))
    inv = (1.0 / np.sqrt(r2.astype(np.float64))).astype(F)
    return x * inv, y * inv


def powers(x, y, re, im):
    """(re + i im), times (x - i y), times (x - i y)^2, ... in FP32."""
    while True:
        yield re, im
        re, im = fma(re, x, im * y), fma(im, x, -(re * y))


def separations(pos, i):
    d = pos[None, :, :] - pos[i][:, None, :]  # FP32, as the kernels subtract
    keep = np.ones(d.shape[:2], bool)
    keep[np.arange(len(i)), i] = False
    return d[keep].reshape(len(i), -1, 3), keep


def lane_sums(v):
    """FP32 sums over the last axis of [n][pairs]: 64 partial sums, then a tree."""
    v = np.pad(v, ((0, 0), (0, -v.shape[1] % 64))).reshape(len(v), -1, 64)
    s = np.zeros((len(v), 64), F)
    for k in range(v.shape[1]):
        s = s + v[:, k]
    while s.shape[1] > 1:
        s = s[:, 0::2] + s[:, 1::2]
    return s[:, 0].astype(np.float64)


def plain_fp32_errors(pos, w, i):
    """rms over primaries i of |S_{m,0} - exact| / rms |S_{m,0}|, m = 0..10."""
    d, keep = separations(pos, i)
    w32 = np.broadcast_to(w.astype(F), keep.shape)[keep].reshape(d.shape[:2])
    x, y = directions(d)
    # the separations themselves carry the rounding of their subtraction
    p64 = pos.astype(np.float64)
    e = (p64[None] - p64[i][:, None])[keep].reshape(d.shape)
    u = e / np.linalg.norm(e, axis=-1, keepdims=True)
    w64 = np.broadcast_to(w, keep.shape)[keep].reshape(d.shape[:2])
    out = []
    for m, (re, im) in zip(range(LMAX + 1), powers(x, y, w32, np.zeros_like(w32))):
        exact = (w64 * (u[..., 0] - 1j * u[..., 1]) ** m).sum(1)
        err = np.abs(lane_sums(re) + 1j * lane_sums(im) - exact)
        out.append(np.sqrt(np.mean(err ** 2) / np.mean(np.abs(exact) ** 2)))
    return np.array(out)


def stored_alm(dev, pos, w, cfg, mask):
    """The a_mm of every primary from the a_lm store, complex [nprim][m]."""
    p, wt = torch.from_numpy(pos).to(dev), torch.from_numpy(w).to(dev)
    mt = torch.from_numpy(mask).to(dev)
    store = api.alm_store(p, wt, cfg)
    api.zeta(p, wt, cfg, primary_mask=mt, alm=store)
    rows = store[256:].view(torch.float64).cpu().numpy().reshape(-1, (LMAX + 1) ** 2)
    rows = rows[:int(mask.sum())]
    cols, off = [], 0
    for m in range(LMAX + 1):  # block m: Re a_lm, l = m.., then (m >= 1) Im a_lm
        nl = LMAX + 1 - m
        cols.append(rows[:, off] + (1j * rows[:, off + nl] if m else 0))
        off += nl if m == 0 else 2 * nl
    return np.stack(cols, 1)


@pytest.mark.parametrize("n,nprim", [(129, 129), (2001, 400), (20001, 200)])
def test_fp32_sums_of_every_m(dev, n, nprim):
    """128, 2000 and 20,000 pairs a primary."""
    say(f"case accuracy by m n={n}")
    pos, w = ball(n, 61)
    mask = np.zeros(n, np.uint8)
    i = np.sort(np.random.default_rng(62).permutation(n)[:nprim])
    mask[i] = 1
    a32 = stored_alm(dev, pos, w, config("fp32"), mask)
    a64 = stored_alm(dev, pos, w, config("fp64"), mask)
    err = np.sqrt(np.mean(np.abs(a32 - a64) ** 2, 0) / np.mean(np.abs(a64) ** 2, 0))
    plain = plain_fp32_errors(pos, w, i)
    for m in range(LMAX + 1):
        say(f"  m={m}: {err[m]:.2e}, plain FP32 {plain[m]:.2e}")
    assert (err <= SLACK * plain).all()


def test_fp32_gradient_at_m_10(dev):
    """The gradient of zeta^10_{10,10}, 400 pairs a galaxy:
    dL/dw_k = |a_k|^2 + sum_i w_i 2 Re(conj(a_i) a_i's term of k)."""
    say("case gradient accuracy")
    n = 401
    pos, w = ball(n, 64)
    gz = np.zeros(api.zeta_shape(LMAX, 1))
    gz[10, 10, 10, 0, 0, 0] = 1.0
    p, wt, g = (torch.from_numpy(a).to(dev) for a in (pos, w, gz))
    # over eight calls: the order of the atomic additions moves the error by a tenth
    g64 = api.zeta_backward(p, wt, config("fp64"), g).cpu().numpy()
    g32 = np.stack([api.zeta_backward(p, wt, config("fp32"), g).cpu().numpy()
                    for _ in range(8)])
    err = np.sqrt(np.mean((g32 - g64) ** 2) / np.mean(g64 ** 2))
    # the same in plain FP32, a_i included (times the square of Y_{10,10}'s factor)
    d, keep = separations(pos, np.arange(n))
    x, y = directions(d)
    p64 = pos.astype(np.float64)
    e = (p64[None] - p64[:, None])[keep].reshape(d.shape)
    u = e / np.linalg.norm(e, axis=-1, keepdims=True)
    c = (u[..., 0] - 1j * u[..., 1]) ** 10
    w2 = np.broadcast_to(w, keep.shape)[keep].reshape(c.shape)
    a = (w2 * c).sum(1)
    zero = np.zeros_like(x)
    for _, (re, im) in zip(range(LMAX + 1), powers(x, y, w2.astype(F), zero)):
        pass
    a32 = lane_sums(re) + 1j * lane_sums(im)
    for _, (re, im) in zip(range(LMAX + 1), powers(x, y, np.ones_like(x), zero)):
        pass
    hr, hi = ((2.0 * v).astype(F)[:, None] for v in (a32.real, a32.imag))
    full, exact = np.zeros((n, n), F), np.zeros((n, n))
    full[keep] = (w.astype(F)[:, None] * fma(re, hr, im * hi)).ravel()
    exact[keep] = (w[:, None] * 2.0 * (a.conj()[:, None] * c).real).ravel()
    s = np.zeros(n, F)
    for j in np.random.default_rng(65).permutation(n):
        s = s + full[j]
    ref = np.abs(a) ** 2 + exact.sum(0)
    plain = np.sqrt(np.mean((np.abs(a32) ** 2 + s - ref) ** 2) / np.mean(ref ** 2))
    say(f"  {err:.2e}, plain FP32 {plain:.2e}")
    assert err <= SLACK * plain
