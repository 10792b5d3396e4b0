"""The wave kernels of the distortion matrix at the edges of their row loop, against
the FP64 oracle: forests of 1 to 9 rows (turns of two or four rows with rows
missing), around the 128 staged rows, and of more pixels than are staged at a time
(256 in the FP32 form); grids with aligned pixels (r_par = 0) and a nonzero lower
edge; few forest pairs, where an FP64 item is one pair.  Repeated launches give the
same sums: rows lost between the two waves of a workgroup would show there.

The short forests take the mean-only projection: the slope term of one or two
pixels is rounding, and the oracle's own two evaluations of it differ by 1e-4.

Tolerances as for the other distortion-matrix tests (1e-12 FP64, 1e-5 FP32, of a
row's largest element); repeats within 1e-12 in both forms, since only the order of
the FP64 additions of the tiles differs."""
import numpy as np
import pytest

import oracle as O
from synth import Grid, concat_realisations, make_patch, uniform_grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}


@pytest.fixture(scope="module")
def lib():
    from paper_2507_00129_amd import Library
    L = Library(0)
    yield L
    L.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("n,npix,model,eta,grid", [
    (14, (1, 9), "log", "mean", uniform_grid(12, 40.0)),
    (6, (126, 131), "log", "mean_slope", uniform_grid(20, 80.0)),
    (5, (250, 262), "lin", "mean_slope", uniform_grid(20, 60.0)),
    (9, (5, 70), "log", "mean_slope", Grid(np.linspace(3.0, 60.0, 14), np.linspace(1.0, 50.0, 21))),
])
def test_turns(lib, prec, variant, n, npix, model, eta, grid):
    from paper_2507_00129_amd import DeviceForests
    F = make_patch(n, 0.35, 17 + n, model=model, npix_range=npix, z_range=(2.1, 2.45))
    ref = O.dmat(F, grid, O.dmat_pairs(F, grid), {"mean": O.MEAN, "mean_slope": O.MEAN_SLOPE}[eta])
    dF = DeviceForests.from_host(F)
    first = None
    for _ in range(3):
        out = lib.dmat(dF, grid, precision=prec, eta=eta, variant=variant, autotune=False)
        D, w = out["dmat"].cpu().numpy(), out["wsum_d"].cpu().numpy()
        if first is None:
            first = (D, w)
            e_d, e_w = O.err_rows(D, ref.D), O.err_rel(w, ref.wd)
            print(f"[{prec} v{variant}] rows={int((ref.wd > 0).sum())} e_D={e_d:.2e} e_W={e_w:.2e}", flush=True)
            assert e_d <= TOL[prec] and e_w <= TOL[prec]
        assert np.abs(D - first[0]).max() <= 1e-12 * np.abs(first[0]).max()
        assert np.abs(w - first[1]).max() <= 1e-12 * np.abs(first[1]).max()


def _spans(F, grid):
    """k_perp rows of each listed forest pair's window, and whether one of its forests
    has at most four pixels and the other at least 64."""
    n_vec = O.unit_vectors(F.ra, F.dec)
    et, out = np.asarray(grid.edges_perp), []
    for f, g in O.dmat_pairs(F, grid):
        s, _ = O.pair_sc(n_vec[f], n_vec[g])
        d = [F.dist[F.forest_slice(k)] for k in (f, g)]
        lo, hi = (min(d[0]) + min(d[1])) * s, (max(d[0]) + max(d[1])) * s
        k0, k1 = np.clip(np.searchsorted(et, [lo, hi], side="right") - 1, 0, len(et) - 2)
        n = sorted(len(x) for x in d)
        out.append((int(k1 - k0 + 1), n[0] <= 4 and n[1] >= 64))
    return out


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("variant", [1, 3])
@pytest.mark.parametrize("grid,blocks", [
    (uniform_grid(40, 150.0, 102, 150.0), (11, 20)),
    (Grid(np.linspace(0.0, 150.0, 21), np.linspace(60.0, 160.0, 202)), (11, 20)),
    (Grid(np.linspace(0.0, 150.0, 8), np.linspace(100.0, 150.0, 586)), (21, 60)),
])
def test_passes_that_leave_a_sweep_without_rows(lib, prec, variant, grid, blocks):
    """Forests of two to four pixels (one turn of the row loop) against long ones in
    windows of several passes: a rectangle pass then has rows of the short forest and
    none of the long one, whose pixels each reach one of the pass's two ranges only.
    The empty sweep has no barrier between the two waves of a workgroup, so it must
    leave the block masks of the turn before it alone."""
    from paper_2507_00129_amd import DeviceForests
    F = concat_realisations([make_patch(n, 2.0, 36 + n, npix_range=npix, z_range=(2.4, 2.7))
                             for n, npix in ((5, (2, 4)), (8, (120, 190)), (6, (2, 4)))])
    F.realisation, F.n_realisations = None, 1  # one survey
    span = [s * (len(grid.edges_par) - 1) for s, mixed in _spans(F, grid) if mixed]
    assert sum(16 * (blocks[0] - 1) < s <= 16 * blocks[1] for s in span) >= 5
    ref = O.dmat(F, grid, O.dmat_pairs(F, grid), O.MEAN)
    # no row that the projection leaves with rounding only (every pair of it in forests
    # whose pixels all fall in that bin): such rows have no relative error
    assert np.abs(ref.D[0]).max(1)[ref.wd[0] > 0].min() > 1e-2
    dF = DeviceForests.from_host(F)
    first = None
    for _ in range(4):
        out = lib.dmat(dF, grid, precision=prec, eta="mean", variant=variant, autotune=False)
        D, w = out["dmat"].cpu().numpy(), out["wsum_d"].cpu().numpy()
        if first is None:
            first = (D, w)
            e_d, e_w = O.err_rows(D, ref.D), O.err_rel(w, ref.wd)
            print(f"[{prec} v{variant}] rows={int((ref.wd > 0).sum())} e_D={e_d:.2e} e_W={e_w:.2e}", flush=True)
            assert e_d <= TOL[prec] and e_w <= TOL[prec]
        assert np.abs(D - first[0]).max() <= 1e-12 * np.abs(first[0]).max()
        assert np.abs(w - first[1]).max() <= 1e-12 * np.abs(first[1]).max()
