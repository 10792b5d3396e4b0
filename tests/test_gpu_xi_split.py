"""How the xi kernel deals out its work and which form it takes, against the FP64
oracle: forests at the edges of the 32-pixel runs and 64-lane blocks, more
neighbours than one item holds, forests whose far end is out of reach (runs of 32
pixels passed over whole), aligned pixel grids (r_par = 0), tickets that are parts
of an item (few forests) and several output slabs with fewer tickets than waves.
The narrow grid's r_par bins are narrower than the pixels, where the rule takes the
form that adds every pair by itself.

Tolerances as for the other xi tests, from the working precision: a bin's sum
within 1e-12 (FP64) or 1e-5 (FP32 products and 32-term sums: 32 x 6e-8 = 2e-6) of
its absolute sum; counts equal."""
import numpy as np
import pytest

import oracle as O
from synth import Grid, concat_realisations, make_patch, sky_cells, uniform_grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}
GRIDS = {"wide": uniform_grid(15, 60.0), "offset": Grid(np.linspace(4.0, 90.0, 12), np.linspace(2.0, 70.0, 18)),
         "narrow": uniform_grid(20, 30.0)}


@pytest.fixture(scope="module")
def lib():
    from paper_2507_00129_amd import Library
    L = Library(0)
    yield L
    L.close()


def compare(out, ref, prec, shape):
    assert ref.n_near_edge == 0, "input has pairs within 1e-12 of an edge; choose another seed"
    np.testing.assert_array_equal(out["npairs"].reshape(shape), ref.npairs.reshape(shape))
    e_n = float(np.max(np.abs(out["num"].reshape(shape) - ref.num.reshape(shape)) /
                       np.where(ref.absnum > 0, ref.absnum, 1.0).reshape(shape)))
    e_w = O.err_rel(out["wsum"].reshape(shape), ref.wsum.reshape(shape))
    print(f"[{prec}] pairs={int(ref.npairs.sum())} e_N={e_n:.2e} e_W={e_w:.2e}", flush=True)
    assert e_n <= TOL[prec] and e_w <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", list(GRIDS))
@pytest.mark.parametrize("n,npix,width", [(3, (64, 65), 0.1), (40, (1, 33), 0.3), (60, (31, 129), 0.5),
                                          (24, (300, 700), 0.6)])
def test_items_runs_and_parts(lib, prec, grid, n, npix, width):
    from paper_2507_00129_amd import DeviceForests
    G = GRIDS[grid]
    # quasars below z = 2.46 start at one wavelength: their pixels are aligned
    log = npix[0] < 200  # 2 Mpc/h pixels; else 0.5
    F = concat_realisations([make_patch(n, width, 40 + n, model="log" if log else "lin", npix_range=npix, z_range=(2.1, 2.6)),
                             make_patch(5, width, 41 + n, npix_range=(1, 40), z_range=(2.1, 2.4))])
    ref = O.xi_sums(F, G)
    out = lib.xi(DeviceForests.from_host(F), G, precision=prec)
    assert lib.last_stats()["variant"] == (1 if grid == "narrow" and log else 3)
    compare({k: out[k].cpu().numpy() for k in ("npairs", "num", "wsum")}, ref, prec, (2, G.n_bins))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,cells", [(9, 3), (60, 5), (150, 2)])
def test_slabs_with_few_tickets(lib, prec, n, cells):
    from paper_2507_00129_amd import DeviceForests
    F = make_patch(n, 0.2 * n ** 0.5, 70 + n, npix_range=(20, 140), z_range=(2.1, 2.6))
    sub, G, n_sub = sky_cells(F, cells, cells), GRIDS["wide"], cells * cells
    ref = O.xi_sums(F, G, sub=sub, n_sub=n_sub)
    out = lib.xi_subsamples(DeviceForests.from_host(F), G, torch.from_numpy(sub).cuda(), n_sub, precision=prec)
    compare({k: out[k].cpu().numpy() for k in ("npairs", "num", "wsum")}, ref, prec, (n_sub, G.n_bins))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", ["wide", "offset", "graded"])
@pytest.mark.parametrize("n,npix,width", [(3, (64, 65), 0.1), (40, (1, 33), 0.3), (60, (127, 130), 0.5)])
def test_gradient_items_and_realisations(lib, prec, grid, n, npix, width):
    """The backward pass over the same edges (lanes own 64 pixels of a forest), one
    realisation and three of unequal size; the gradients within the forward's
    tolerances of their largest value."""
    from paper_2507_00129_amd import DeviceForests
    G = GRIDS[grid] if grid != "graded" else Grid(np.linspace(0.0, 60.0, 11), 60.0 * (np.arange(13) / 12) ** 1.3)
    one = make_patch(n, width, 40 + n, npix_range=npix, z_range=(2.1, 2.6))
    for F in (one, concat_realisations([one, make_patch(7, width, 41 + n, npix_range=(1, 40), z_range=(2.1, 2.4)),
                                        make_patch(33, width, 42 + n, npix_range=(60, 70), z_range=(2.1, 2.4))])):
        X = O.xi_sums(F, G)
        assert X.n_near_edge == 0, "input has pairs within 1e-12 of an edge; choose another seed"
        gxi = np.random.default_rng(n).normal(size=X.xi.shape)
        want = O.xi_grad(F, G, gxi, X.xi, X.wsum)
        dF = DeviceForests.from_host(F)
        put = lambda x: torch.as_tensor(x, device="cuda:0")
        got = lib.xi_backward(dF, G, put(gxi), put(X.xi), put(X.wsum), precision=prec)
        for g, w in zip(got, want):
            e = O.err_norm(g.cpu().numpy(), w)
            print(f"[{prec} {grid}] e_g={e:.2e}", flush=True)
            assert e <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_par,n_perp", [(58, 60), (60, 60), (263, 14)])
def test_bin_means_that_fill_the_lds(lib, prec, n_par, n_perp):
    """Bin means over 3480, 3600 and 3682 bins: below and above the line where the
    sums leave room for items of two neighbours and one entry for the pairs outside."""
    from paper_2507_00129_amd import DeviceForests
    G = uniform_grid(n_par, 150.0, n_perp, 40.0)
    F = make_patch(40, 0.6, 5, npix_range=(1, 140), z_range=(2.1, 2.6))
    ref = O.xi_sums(F, G)
    out = lib.xi_means(DeviceForests.from_host(F), G, precision=prec)
    compare({k: out[k].cpu().numpy() for k in ("npairs", "num", "wsum")}, ref, prec, (1, G.n_bins))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_par,n_perp", [(58, 60), (60, 60), (263, 14), (14, 263)])
def test_bin_mean_coordinates_that_fill_the_lds(lib, prec, n_par, n_perp):
    """The coordinates of the same bin means, the sums that only this form has.  A mean
    is off by the coordinates' rounding in the working precision u (as bounded for the
    FP32 edge guard, in bins: (2 M / dr + 3 (N + 2)) u and ((3 M + 2 D) s / dr + N + 2) u)
    and by that of the runs of 32 terms of up to N in both sums (64 N u); the FP64
    additions of the runs of a bin of n pairs add some sqrt(n) 2^-53 N."""
    from paper_2507_00129_amd import DeviceForests
    G = uniform_grid(n_par, 150.0, n_perp, 40.0)
    F = make_patch(40, 0.6, 5, npix_range=(1, 140), z_range=(2.1, 2.6))
    ref = O.xi_sums(F, G, means=True)
    out = {k: v.cpu().numpy() for k, v in lib.xi_means(DeviceForests.from_host(F), G, precision=prec).items()}
    np.testing.assert_array_equal(out["npairs"], ref.npairs)
    u = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24}[prec]
    acc = 8.0 * 2.0 ** -53 * float(ref.npairs.max()) ** 0.5
    lo, hi = F.dist.min(), F.dist.max()
    M, D, s = 0.5 * (hi - lo), 0.5 * (hi + lo), 40.0 / (2.0 * lo)
    dp, dt = 150.0 / n_par, 40.0 / n_perp
    tol_p = u * (2.0 * M / dp + 67.0 * (n_par + 2)) + acc * n_par
    tol_t = u * ((3.0 * M + 2.0 * D) * s / dt + 65.0 * (n_perp + 2)) + acc * n_perp
    tol_z = 70.0 * u + acc
    for got, want, scale, tol in zip((out["rpar"], out["rperp"], out["z"]), O.bin_means(ref),
                                     (dp, dt, 1.0), (tol_p, tol_t, tol_z)):
        e = float(np.max(np.abs(got - want))) / scale
        print(f"[{prec} {n_par}x{n_perp}] e={e:.2e} of {tol:.2e}", flush=True)
        assert e <= tol and np.abs(want).max() > 0.0


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("per_bin,variant", [(0.97, 1), (1.12, 3), (1.5, 3)])
def test_form_by_pixels_per_bin(lib, prec, per_bin, variant):
    """Runs from 1.05 pixels to an r_par bin on, single pairs below."""
    from paper_2507_00129_amd import DeviceForests
    F = make_patch(30, 0.5, 77, npix_range=(20, 120), z_range=(2.1, 2.6))
    first, last = F.offsets[:-1], F.offsets[1:] - 1
    spacing = float(np.sum(F.dist[last] - F.dist[first]) / (F.n_pix - F.n_forests))
    G = uniform_grid(25, 25 * per_bin * spacing, 12, 40.0)
    out = lib.xi(DeviceForests.from_host(F), G, precision=prec)
    assert lib.last_stats()["variant"] == variant
    compare({k: out[k].cpu().numpy() for k in ("npairs", "num", "wsum")}, O.xi_sums(F, G), prec, (1, G.n_bins))
