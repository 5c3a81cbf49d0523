"""NaN and infinities in the vectors of applies and of the signal filter.

A row tile (16 outputs of a position) with a nonzero table entry for such a value meets it; in its
other rows the product is 0 times that value.  An output with a nonzero entry for a NaN is NaN; one
with a nonzero entry for an infinity, whose tile meets no other such value, is that infinity times
the entry's sign.  Outputs in tiles that meet none are the sums of the finite values.  The filter's
outputs further than its taps reach from such a sample are those of the samples within reach.

Tolerances: those of the finite sums, as derived where the tile edges are tested."""
import numpy as np
import pytest

from oracle import filters as ofil
from oracle import operators as oops
import workloads as W
from test_gpu_apply_shapes import odd_start, on_scan, random_table

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402


def wide_table(rng, nz, nt, K):
    """Columns at forty offsets of a wide footprint."""
    full = random_table(rng, nz, nt, 2)
    H = np.zeros((2 * K + 1, 2 * K + 1, nz, nt))
    for i in range(40):
        H[rng.integers(0, 2 * K + 1), rng.integers(0, 2 * K + 1)] = full[i % 5, 1 + i % 4]
    return H


def tiles(hit):
    """Every row of the 16-row tiles in which `hit` holds somewhere."""
    n = hit.shape[2]
    pad = np.pad(hit, ((0, 0), (0, 0), (0, -n % 16)))
    return np.repeat(pad.reshape(*hit.shape[:2], -1, 16).any(3), 16, axis=2)[..., :n]


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", [(9, 33, 33, 95, 4), (13, 30, 48, 129, 6), (70, 130, 10, 600, 37)],
                         ids=lambda g: "x".join(map(str, g)))
def test_applies_keep_nonfinite_values_where_the_table_meets_them(grid, dtype):
    ny, nx, nz, nt, K = grid
    rng = np.random.default_rng(nt)
    H = wide_table(rng, nz, nt, K) if K > 20 else random_table(rng, nz, nt, K)
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    tdt, u = (torch.float64, 2.0 ** -53) if dtype == "fp64" else (torch.float32, 2.0 ** -24)
    npt = np.float64 if dtype == "fp64" else np.float32
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32")) as m:
        for name in ("forward", "adjoint"):
            op, n_in = getattr(oops, name), nz if name == "forward" else nt
            v = rng.standard_normal((ny, nx, n_in)).astype(npt)
            spots = {k: (int(rng.integers(ny)), int(rng.integers(nx)), int(rng.integers(n_in)))
                     for k in ("nan", "inf", "-inf")}
            finite, hit = v.copy(), {}
            for k, at in spots.items():
                v[at], finite[at] = float(k), 0
                one = np.zeros(v.shape)
                one[at] = 1
                hit[k] = on_scan(op, H, one)  # the table entry of the value in each output
            print(f"[non-finite {grid} {dtype} {name}]", flush=True)
            got = getattr(m, name)(odd_start(v, tdt), dtype).cpu().numpy().astype(np.float64)
            met = {k: tiles(h != 0) for k, h in hit.items()}  # the row tiles that meet the value
            nan = hit["nan"] != 0
            assert np.isnan(got[nan]).all()
            for k, other in (("inf", "-inf"), ("-inf", "inf")):
                sure = (hit[k] != 0) & ~met["nan"] & ~met[other]
                assert np.array_equal(got[sure], float(k) * np.sign(hit[k][sure]))
            ref = on_scan(op, H, finite.astype(np.float64))
            terms = on_scan(op, (H != 0).astype(np.float64), np.ones(v.shape)).max()
            bound = (2 * np.sqrt(terms) + 8) * u * on_scan(op, np.abs(H),
                                                           np.abs(finite).astype(np.float64))
            tile = met["nan"] | met["inf"] | met["-inf"]
            assert tile.any() and not tile.all()
            assert np.all(np.abs(got - ref)[~tile] <= bound[~tile])


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("grid", [(9, 33, 33, 95, 4), (13, 30, 48, 129, 6), (20, 40, 70, 200, 3)],
                         ids=lambda g: "x".join(map(str, g)))
def test_reduced_precision_spreads_nonfinite_values_no_further_than_runs(grid, dtype):
    """FP8 applies multiply runs of eight entries by row tiles of 16: a non-finite entry, which has
    the NaN code, reaches the outputs of tiles with a nonzero table entry for its run, and no others.
    In BF16 those with one for the entry itself, and an infinity times a nonzero entry is one."""
    ny, nx, nz, nt, K = grid
    rng = np.random.default_rng(nt + K)
    H = random_table(rng, nz, nt, K)
    H[:, :, ::3] = 0  # runs and offsets without entries, so that bundles are filled up
    H[rng.random(H.shape[:2]) < 0.6] = 0
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32", dtype)) as m:
        for name in ("forward", "adjoint"):
            op, n_in = getattr(oops, name), nz if name == "forward" else nt
            for value in (np.nan, np.inf):
                v = rng.standard_normal((ny, nx, n_in)).astype(np.float32)
                at = (int(rng.integers(ny)), int(rng.integers(nx)), int(rng.integers(n_in)))
                v[at] = value
                run, one = np.zeros(v.shape), np.zeros(v.shape)
                run[at[0], at[1], at[2] // 8 * 8:at[2] // 8 * 8 + 8] = 1
                one[at] = 1
                hit = on_scan(op, H, one)
                print(f"[non-finite {grid} {dtype} {name} {value}]", flush=True)
                got = getattr(m, name)(torch.from_numpy(v).cuda(), dtype).cpu().numpy()
                bad = ~np.isfinite(got)
                assert bad[hit != 0].all()
                met = tiles(on_scan(op, (H != 0).astype(np.float64), run) != 0)
                if dtype == "bf16":
                    met = tiles(hit != 0)
                    if value == np.inf:
                        assert np.array_equal(got[hit != 0], np.sign(hit[hit != 0]) * np.inf)
                assert not met.all() and not bad[~met].any()


@pytest.mark.parametrize("nt,L", [(64, 5), (257, 16), (40, 0)])
def test_filter_spreads_a_nonfinite_sample_no_further_than_its_taps(nt, L):
    cfg = W.config("tiny")
    g = W.grid(5, 10e-6, 2, 10e-6, nt, 0, 0, ny=3)
    f = dict(f_lo_hz=0.5e6, f_hi_hz=80e6, half_taps=L)
    h = ofil.bandpass_taps(f["f_lo_hz"], f["f_hi_hz"], g["fs_hz"], L)
    rng = np.random.default_rng(nt)
    with P.Model(cfg["sensor"], g, dtypes=("fp64", "fp32"), filter=f) as m:
        for npt, u in ((np.float64, 2.0 ** -53), (np.float32, 2.0 ** -24)):
            v = rng.standard_normal((3, 5, nt)).astype(npt)
            ref = ofil.filter_time(v.astype(np.float64), h)
            bound = (2 * np.sqrt(2 * L + 1) + 8) * u * ofil.filter_time(np.abs(v).astype(np.float64),
                                                                        np.abs(h))
            at = rng.integers(0, nt, (3, 5))
            bad = np.where(rng.random((3, 5)) < 0.5, np.nan, np.inf).astype(npt)
            np.put_along_axis(v, at[..., None], bad[..., None], axis=2)
            print(f"[filter, non-finite nt {nt} L {L} {npt.__name__}]", flush=True)
            got = m.filter_signals(torch.from_numpy(v).cuda()).cpu().numpy().astype(np.float64)
            reached = np.abs(np.arange(nt) - at[..., None]) <= L
            inner = np.abs(np.arange(nt) - at[..., None]) <= max(0, L - 1)  # the outer taps may be 0
            assert not np.isfinite(got[inner]).any()
            assert np.all(np.abs(got - ref)[~reached] <= bound[~reached])
