"""Small catalogues of a batch, which go through the stages in groups: each zeta is
bitwise that of a separate call, whether or not the pairs are asked for."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1709_00086_amd import api, catalogues as C

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("sizes,lmax,nbins", [
    ([8192, 7000, 0, 16384, 3, 16385, 129], 10, 10),  # more blocks than one launch has room for
    ([700, 1500, 2500] * 7, 10, 6),                    # more catalogues than a group
    ([5000, 128, 6144, 6145, 127], 2, 3),              # one macro tile an m
])
def test_grouped_catalogues_bitwise(dev, sizes, lmax, nbins, precision, masked):
    say(f"case grouped bits {len(sizes)} lmax={lmax} nbins={nbins} {precision} masked={masked}")
    L, rmax = 400.0, 40.0
    pos, w, offs = C.mock_batch(sizes, L, 93)
    mask = (np.random.default_rng(94).uniform(size=len(w)) < 0.6).astype(np.uint8)
    cfg = api.Config(box=(L, L, L), rmax=rmax, nbins=nbins, lmax=lmax, precision=precision,
                     basis="spin")
    pt, wt, mt = (torch.from_numpy(a).to(dev) for a in (pos, w, mask))
    if not masked:
        mt = None
    z = api.zeta_batch(pt, wt, cfg, offs, primary_mask=mt)
    zp, _ = api.zeta_batch(pt, wt, cfg, offs, primary_mask=mt, return_pairs=True)
    assert torch.equal(z, zp)
    for c, n in enumerate(sizes):
        a, b = int(offs[c]), int(offs[c + 1])
        if n == 0:
            assert not z[c].any()
            continue
        one = api.zeta(pt[a:b].contiguous(), wt[a:b].contiguous(), cfg,
                       primary_mask=None if mt is None else mt[a:b].contiguous())
        assert torch.equal(z[c], one), c


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("basis", ["spin", "cartesian"])
def test_grouped_catalogues_and_oracle(dev, basis, precision):
    """FP64 1e-10, FP32 1e-5 of max|zeta|."""
    say(f"case grouped oracle {basis} {precision}")
    L, rmax, nbins, lmax = 300.0, 60.0, 6, 10
    sizes = [900, 0, 1, 2, 1500, 700]
    pos, w, offs = C.mock_batch(sizes, L, 91)
    cfg = api.Config(box=(L, L, L), rmax=rmax, nbins=nbins, lmax=lmax, precision=precision,
                     basis=basis)
    z = api.zeta_batch(torch.from_numpy(pos).to(dev), torch.from_numpy(w).to(dev), cfg,
                       offs).cpu().numpy()
    for c in (0, 4):
        a, b = int(offs[c]), int(offs[c + 1])
        cat = C.Catalogue(name=f"batch{c}", pos=pos[a:b], w=w[a:b], box=(L, L, L), rmax=rmax,
                          nbins=nbins, lmax=lmax, los="z", observer=(0.0, 0.0, 0.0),
                          periodic=True, box_lo=(0.0, 0.0, 0.0))
        ref = oracle.zeta(cat)
        err = np.abs(z[c] - ref).max() / np.abs(ref).max()
        say(f"  catalogue {c}: max|dzeta|/max|zeta| = {err:.2e}")
        assert err <= (1e-10 if precision == "fp64" else 1e-5)
    for c in (1, 2):
        assert not z[c].any()
