"""How the work is cut up must not change the results.
FP64 against the oracle (1e-10 of max|zeta|); the FP32 and BF16x3 zeta stages
against the FP64 zeta stage on the same FP32 pairs (1e-5)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1709_00086_amd import api, catalogues as C

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 1e-5}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def cfg_of(cat, precision, basis="spin", **kw):
    return api.Config(box=cat.box, rmax=cat.rmax, nbins=cat.nbins, lmax=cat.lmax, los=cat.los,
                      observer=cat.observer, periodic=cat.periodic, box_lo=cat.box_lo,
                      precision=precision, basis=basis, **kw)


def on(dev, cat):
    return (torch.from_numpy(np.ascontiguousarray(cat.pos)).to(dev),
            torch.from_numpy(np.ascontiguousarray(cat.w)).to(dev))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("count", [1, 127, 128, 129, 2100, 6000])
def test_gram_blocks_hold_any_number_of_primaries(dev, precision, count):
    """Primaries fewer than, just over and many times the least rows of a block
    (128), of a catalogue whose launch covers 6000.  (The oracle is no reference
    for FP32 pairs here: with 59 pairs a primary, a pair or two that FP32 puts
    into the next shell already moves zeta by 4e-5.)"""
    say(f"case gram blocks {count} {precision}")
    cat = C.uniform(6000, 300.0, seed=71, dtype=np.float64, weights="uniform", rmax=40.0)
    mask = C.primary_mask(cat.n, count, seed=72)
    pos, w = on(dev, cat)
    mt = torch.from_numpy(mask).to(dev)
    z = api.zeta(pos, w, cfg_of(cat, precision), primary_mask=mt).cpu().numpy()
    if precision == "fp64":
        ref = oracle.zeta(cat, primary_mask=mask)
    else:
        ref = api.zeta(pos, w, cfg_of(cat, precision, zeta_precision="fp64"),
                       primary_mask=mt).cpu().numpy()
    e = np.abs(z - ref).max() / np.abs(ref).max()
    say(f"  max|dz|/max|z| = {e:.2e}")
    assert e <= TOL[precision]


@pytest.mark.parametrize("los", ["z", "observer"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lmax", [0, 3, 4, 5, 6, 7, 8, 9, 10])
def test_every_degree_of_the_spin_kernels(dev, lmax, precision, los):
    """zeta, the distinct zeta and the gradient at each l_max, on both sides of
    the kernels' degrees 4, 6, 8 and 10.  Float32 positions and no pair within
    1e-4 of a shell edge, so that FP32 puts every pair into the oracle's shell;
    tolerances: FP64 1e-10, FP32 1e-5 of max|zeta| and 1e-4 of max|gradient|."""
    say(f"case degree lmax={lmax} {precision} {los}")
    cat = C.tiny(n=300, L=150.0, seed=75, rmax=45.0, nbins=5, lmax=lmax, periodic=(los == "z"),
                 los=los, dtype=np.float32, observer=(-100.0, 20.0, -50.0))
    pos, w = on(dev, cat)
    cfg = cfg_of(cat, precision)
    tol = TOL[precision]
    for distinct in (False, True):
        c = cfg_of(cat, precision, distinct=distinct)
        z, pairs = api.zeta(pos, w, c, return_pairs=True)
        ref, pairs_ref = oracle.zeta(cat, distinct=distinct, return_pairs=True)
        e = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"  distinct={distinct}: max|dz|/max|z| = {e:.2e}")
        assert pairs == pairs_ref
        assert e <= tol
    gz = C.loss_weights(lmax, cat.nbins, seed=76)
    g = api.zeta_backward(pos, w, cfg, torch.from_numpy(gz).to(dev)).cpu().numpy()
    gref = oracle.grad(cat, gz)
    e = np.abs(g - gref).max() / np.abs(gref).max()
    say(f"  gradient: {e:.2e}")
    assert e <= (1e-10 if precision == "fp64" else 1e-4)


def clump(seed, n=3000, L=300.0, k=400):
    """k galaxies within 2 Mpc/h of each other in a sparse periodic box."""
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, L, size=(n, 3))
    pos[:k] = np.array([150.0, 140.0, 160.0]) + rng.uniform(-1.0, 1.0, size=(k, 3))
    return C.Catalogue("clump", pos.astype(np.float32), rng.uniform(0.5, 1.5, size=n), (L,) * 3,
                       (0.0,) * 3, True, 60.0, 6, 10, "z")


@pytest.mark.parametrize("basis", ["spin", "cartesian"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_shells_searched_together_and_their_overflow(dev, precision, basis):
    """A sparse catalogue, whose shells are searched together into a list of 224
    (FP32) or 128 pairs, with a clump whose primaries have 399 pairs in the first
    shell: pair counts, zeta, the distinct zeta and the gradient.  Float32
    positions and no pair within 1e-5 of a shell edge; tolerances: FP64 1e-10,
    FP32 1e-5 of max|zeta| and 1e-4 of max|gradient|."""
    say(f"case clump {precision} {basis}")
    cat = clump(81)
    pos, w = on(dev, cat)
    for distinct in (False, True):
        z, pairs = api.zeta(pos, w, cfg_of(cat, precision, basis, distinct=distinct),
                            return_pairs=True)
        ref, pairs_ref = oracle.zeta(cat, distinct=distinct, return_pairs=True)
        e = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"  distinct={distinct}: pairs {pairs} ({pairs_ref}), max|dz|/max|z| = {e:.2e}")
        assert pairs == pairs_ref
        assert e <= TOL[precision]
    gz = C.loss_weights(cat.lmax, cat.nbins, seed=78)
    g = api.zeta_backward(pos, w, cfg_of(cat, precision, basis),
                          torch.from_numpy(gz).to(dev)).cpu().numpy()
    gref = oracle.grad(cat, gz)
    e = np.abs(g - gref).max() / np.abs(gref).max()
    say(f"  gradient: {e:.2e}")
    assert e <= (1e-10 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 6143, 6144, 6145])
@pytest.mark.parametrize("masked", [False, True])
def test_cell_stage_of_small_catalogues(dev, n, masked):
    """The cell stage of one workgroup (up to 6144 galaxies) and the general one:
    pair counts and zeta against the oracle (FP64, 1e-10), a third of the galaxies
    in one clump so that cells are empty and crowded."""
    say(f"case cell stage n={n} masked={masked}")
    rng = np.random.default_rng(83)
    pos = rng.uniform(0.0, 200.0, size=(n, 3))
    pos[: n // 3] = 90.0 + rng.normal(0.0, 2.0, size=(n // 3, 3))
    cat = C.Catalogue("cells", pos, rng.uniform(0.5, 1.5, size=n), (200.0,) * 3, (0.0,) * 3, True,
                      20.0, 3, 4, "z")
    mask = (rng.uniform(size=n) < 0.4).astype(np.uint8) if masked else None
    p, w = on(dev, cat)
    z, pairs = api.zeta(p, w, cfg_of(cat, "fp64"), return_pairs=True,
                        primary_mask=None if mask is None else torch.from_numpy(mask).to(dev))
    ref, pairs_ref = oracle.zeta(cat, primary_mask=mask, return_pairs=True)
    e = np.abs(z.cpu().numpy() - ref).max()
    say(f"  pairs {pairs}, max|dz| = {e:.2e} of {np.abs(ref).max():.2e}")
    assert pairs == pairs_ref
    assert e <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("n,nregions,distinct", [(7, 12, False), (1500, 1, True),
                                                 (1500, 300, False), (1500, 1499, True)])
def test_regions_in_one_pass(dev, n, nregions, distinct):
    """Region ids outside the range and a mask; more regions than galaxies, and
    more than one digit of the sort.  Each region's zeta against the oracle with
    the region as the mask (FP64, 1e-10 of max|zeta| over all of them)."""
    say(f"case regions n={n} R={nregions} distinct={distinct}")
    cat = C.tiny(n=n, L=150.0, seed=87, rmax=40.0, nbins=3, lmax=3)
    rng = np.random.default_rng(88)
    region = rng.integers(-2, nregions + 2, size=n).astype(np.int32)
    mask = (rng.uniform(size=n) < 0.7).astype(np.uint8)
    pos, w = on(dev, cat)
    z = api.zeta_regions(pos, w, cfg_of(cat, "fp64", distinct=distinct),
                         torch.from_numpy(region).to(dev), nregions,
                         primary_mask=torch.from_numpy(mask).to(dev)).cpu().numpy()
    refs = {r: oracle.zeta(cat, primary_mask=((region == r) & (mask != 0)).astype(np.uint8),
                           distinct=distinct)
            for r in sorted({0, nregions // 2, nregions - 1, min(6, nregions - 1)})}
    scale = max(np.abs(v).max() for v in refs.values())
    for r, ref in refs.items():
        assert np.abs(z[r] - ref).max() <= 1e-10 * scale, r
    every = oracle.zeta(cat, primary_mask=((region >= 0) & (region < nregions) &
                                           (mask != 0)).astype(np.uint8), distinct=distinct)
    e = np.abs(z.sum(0) - every).max() / max(np.abs(every).max(), 1e-300)
    say(f"  sum over regions: {e:.2e}")
    assert e <= 1e-10


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("lmax,nbins", [(0, 1), (0, 16), (0, 17), (0, 32), (1, 8), (3, 32),
                                        (9, 13), (10, 6), (10, 32)])
def test_gram_macro_tiles_of_any_width(dev, precision, lmax, nbins):
    """Blocks C_m of 1 to 640 columns: one tile, one past a tile, an odd number of
    tiles, exactly one panel of 128, one past it, several."""
    say(f"case gram widths lmax={lmax} nbins={nbins} {precision}")
    cat = C.uniform(300, 100.0, seed=73, dtype=np.float64, weights="uniform", rmax=45.0,
                    nbins=nbins, lmax=lmax)
    pos, w = on(dev, cat)
    z = api.zeta(pos, w, cfg_of(cat, precision)).cpu().numpy()
    if precision == "fp64":
        ref = oracle.zeta(cat)
    else:
        ref = api.zeta(pos, w, cfg_of(cat, precision, zeta_precision="fp64")).cpu().numpy()
    e = np.abs(z - ref).max() / np.abs(ref).max()
    say(f"  max|dz|/max|z| = {e:.2e}")
    assert e <= TOL[precision]


@pytest.mark.parametrize("nregions", [2, 40, 70])
def test_regions_of_very_different_sizes(dev, nregions):
    """One region holds nearly all galaxies (many Gram blocks), others a few or
    none; more regions than one launch of the Gram products takes.  FP64, 1e-10 of
    the largest zeta."""
    say(f"case uneven regions {nregions}")
    n = 4000
    cat = C.uniform(n, 250.0, seed=75, dtype=np.float64, weights="uniform", rmax=30.0, nbins=4,
                    lmax=4)
    rng = np.random.default_rng(76)
    region = np.full(n, nregions // 2, dtype=np.int32)
    few = rng.choice(n, size=600, replace=False)
    region[few] = rng.integers(0, nregions, size=600)
    region[region == nregions - 1] = 0  # the last one holds none
    pos, w = on(dev, cat)
    z = api.zeta_regions(pos, w, cfg_of(cat, "fp64"), torch.from_numpy(region).to(dev),
                         nregions).cpu().numpy()
    scale = np.abs(z).max()
    for r in sorted({0, nregions // 2, nregions - 2, nregions - 1}):
        ref = oracle.zeta(cat, primary_mask=(region == r).astype(np.uint8))
        assert np.abs(z[r] - ref).max() <= 1e-10 * scale, r
    assert not z[nregions - 1].any()


@pytest.mark.parametrize("precision,basis", [("fp64", "spin"), ("fp32", "spin"),
                                             ("fp64", "cartesian")])
@pytest.mark.parametrize("sizes", [[300, 200], [1, 0, 63, 64, 0, 65, 2], [700] * 20,
                                   [16383, 16384, 16385, 40, 3000]])
@pytest.mark.parametrize("masked", [False, True])
def test_catalogues_of_a_batch_together(dev, sizes, masked, precision, basis):
    """Fewest and more catalogues than a group holds, empty ones, and the sizes
    around its largest.  Each against a call of its own (FP64 1e-10, FP32 1e-5 of
    max|zeta|), with a mask that leaves some without primaries."""
    say(f"case batch {sizes} {masked} {precision} {basis}")
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    cat = C.uniform(int(off[-1]), 300.0, seed=77, dtype=np.float64, weights="uniform",
                    rmax=30.0, nbins=4, lmax=5)
    mask = (np.random.default_rng(78).uniform(size=cat.n) < 0.3).astype(np.uint8)
    mask[:off[1]] = 0
    pos, w = on(dev, cat)
    mt = torch.from_numpy(mask).to(dev) if masked else None
    cfg = cfg_of(cat, precision, basis=basis)
    z = api.zeta_batch(pos, w, cfg, off, primary_mask=mt).cpu().numpy()
    scale = np.abs(z).max()
    for c, n in enumerate(sizes):
        a, b = int(off[c]), int(off[c + 1])
        if n == 0:
            assert not z[c].any()
            continue
        ref = api.zeta(pos[a:b], w[a:b], cfg,
                       primary_mask=mt[a:b].contiguous() if masked else None).cpu().numpy()
        assert np.abs(z[c] - ref).max() <= (1e-10 if precision == "fp64" else 1e-5) * scale, c
