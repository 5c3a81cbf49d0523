"""Scratch memory of applies and solves: FP64 and FP32 applies read the caller's vector, so a scan
whose tiles are not cut needs none."""
import math

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
def test_solve_of_an_uncut_scan_holds_its_vectors_and_no_stage(dtype):
    """LSQR holds u and a signal vector, v, w and an image vector, and a few KB of sums and scalars;
    FISTA one signal vector and four images.  The solves run within that."""
    cfg = W.config("tiny")
    g = dict(cfg["grid"], nx=300, ny=300, nz=48, nt=48)
    size = 8 if dtype == "fp64" else 4
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    with P.Model(cfg["sensor"], g, dtypes=("fp64", "fp32")) as m:
        info, d = m.info(), P.DTYPES[dtype]
        assert info["pieces"][d] == info["row_tiles"][d]
        assert info["pieces_adj"][d] == info["row_tiles_adj"][d]
        s, x = size * math.prod(m.signal_shape), size * math.prod(m.image_shape)
        lsqr = P.aroam_solve_footprint(m.handle, 0, lam=1.0, iters=2, inner=d, outer=d)
        fista = P.aroam_solve_footprint(m.handle, 1, lam=1.0, iters=2, inner=d, outer=d)
        assert 2 * s + 3 * x <= lsqr <= 2 * s + 3 * x + (64 << 10)
        assert s + 4 * x <= fista <= s + 4 * x + (64 << 10)
        y = m.forward(torch.randn(m.image_shape, device="cuda", dtype=tdt), dtype)
        assert torch.isfinite(y).all()
        for solve in (m.solve_lsqr, m.solve_l1):
            out, _ = solve(y, iters=2, inner=dtype, outer=dtype)
            assert torch.isfinite(out).all()
