"""Applies at the edges of the kernels' tilings, against the oracle's operators on a random
table.

Each grid sits at an edge of the tiles: one position, fewer positions than a 16-position tile,
one more than a tile or a patch, patches whose second tile column is empty, inner lengths of
one, just below, at and above a run, a chunk and a row tile, offsets reaching beyond the whole
scan.  The table's windows are random (empty columns among them), so that tiles, runs and
bundles are cut in every way.  The vectors start at an odd element of their storage, so that
their rows are aligned to nothing more than an element.

Tolerance: an output is a sum of n products; with unit roundoff u (2^-53, 2^-24) the errors of
the partial sums grow like sqrt(n) u times the sum of the absolute products, and the bound takes
twice that plus 8 u for the roundings of the table and of single products."""
import numpy as np
import pytest

from oracle import operators as oops

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402

# (ny, nx, nz, nt, K)
GRIDS = [(1, 1, 1, 5, 0), (1, 1, 40, 70, 3), (2, 15, 7, 33, 1), (3, 17, 8, 31, 2),
         (5, 16, 16, 64, 3), (4, 32, 17, 65, 2), (9, 33, 33, 95, 4), (8, 49, 31, 66, 5),
         (13, 30, 48, 129, 6), (3, 65, 25, 48, 9), (17, 20, 9, 150, 12)]


def random_table(rng, nz, nt, K):
    W = 2 * K + 1
    H = np.zeros((W, W, nz, nt))
    lo = rng.integers(0, nt, (W, W, nz))
    hi = np.minimum(nt - 1, lo + rng.integers(0, 45, (W, W, nz)))
    on = rng.random((W, W, nz)) < 0.8
    n = np.arange(nt)
    inside = on[..., None] & (n >= lo[..., None]) & (n <= hi[..., None])
    H[inside] = rng.standard_normal(int(inside.sum()))
    return H


def on_scan(op, H, v):
    """The oracle's operator on a scan that may be smaller than the offsets reach: the scan is
    continued by zeros to K + 1 positions and the result cut back."""
    ny, nx, K = v.shape[0], v.shape[1], (H.shape[0] - 1) // 2
    pad = ((0, max(0, K + 1 - ny)), (0, max(0, K + 1 - nx)), (0, 0))
    return op(H, np.pad(v, pad))[:ny, :nx]


def odd_start(a, dtype):
    """The array on the GPU, one element into its storage."""
    t = torch.empty(a.size + 1, dtype=dtype, device="cuda")[1:].view(a.shape)
    t.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return t


def check(H, ny, nx, dtype, rng, ops=("forward", "adjoint")):
    K, (nz, nt) = (H.shape[0] - 1) // 2, H.shape[2:]
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    tdt, u = (torch.float64, 2.0 ** -53) if dtype == "fp64" else (torch.float32, 2.0 ** -24)
    npt = np.float64 if dtype == "fp64" else np.float32
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32")) as m:
        for name in ops:
            op, shape = getattr(oops, name), (ny, nx, nz if name == "forward" else nt)
            v = rng.standard_normal(shape).astype(npt)
            print(f"[{(ny, nx, nz, nt, K)} {dtype} {name}]", flush=True)
            got = getattr(m, name)(odd_start(v, tdt), dtype).cpu().numpy().astype(np.float64)
            ref = on_scan(op, H, v.astype(np.float64))
            terms = on_scan(op, (H != 0).astype(np.float64), np.ones(shape)).max()
            bound = (2 * np.sqrt(terms) + 8) * u * on_scan(op, np.abs(H),
                                                           np.abs(v).astype(np.float64))
            assert np.all(np.abs(got - ref) <= bound)


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_apply_matches_oracle_at_tile_edges(grid, dtype):
    ny, nx, nz, nt, K = grid
    rng = np.random.default_rng(1000 * ny + nx)
    check(random_table(rng, nz, nt, K), ny, nx, dtype, rng)


@pytest.mark.parametrize("grid", [(3, 5, 9, 20, 97), (2, 40, 5, 33, 62), (61, 120, 8, 512, 37)],
                         ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
def test_wide_footprints(grid, dtype):
    """The widest footprint, one that leaves a single workgroup per CU, and one whose FP32 forward
    owns patches of eight rows; a table with columns at a few dozen offsets, corners included."""
    ny, nx, nz, nt, K = grid
    rng = np.random.default_rng(K)
    full = random_table(rng, nz, nt, 2)
    H = np.zeros((2 * K + 1, 2 * K + 1, nz, nt))
    lim = (min(K, ny - 1), min(K, nx - 1))
    for i, (a, b) in enumerate([(K, K), (0, 0), (2 * K, 0), (K + lim[0], K - lim[1])]):
        H[a, b] = full[i, 0]
    for i in range(40):
        a = K + rng.integers(-lim[0], lim[0] + 1)
        b = K + rng.integers(-lim[1], lim[1] + 1)
        H[a, b] = full[i % 5, 1 + i % 4]
    check(H, ny, nx, dtype, rng)
