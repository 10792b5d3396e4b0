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
from synth import Grid, make_patch, uniform_grid

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
