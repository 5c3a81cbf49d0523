"""Scratch memory of applies and solves: FP64 and FP32 applies read the caller's vector, so a scan
whose tiles are not cut needs none; the allocation-free forward takes every BF16 and FP8 scan whose
padded input (for FP8 with its scales) fits its 64 MiB, whatever the cut of the launch needs."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402
from test_gpu_apply_shapes import random_table  # noqa: E402
from test_zz_no_alloc import _raw  # noqa: E402


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


@pytest.mark.parametrize("dtype,ny,nz,fits", [
    ("bf16", 16, 65536, True),    # 16 x 32 x 65536 x 2 bytes: the array to the byte
    ("bf16", 16, 64000, True),    # 1.5 MiB left for slots
    ("bf16", 24, 65536, False),
    ("fp8", 32, 63488, True),     # 62 MiB and 992 x 514 x 4 bytes of scales
    ("fp8", 32, 64512, False),    # 63 MiB and 2.0 of scales
])
def test_noalloc_forward_takes_every_input_that_fits(dtype, ny, nz, fits):
    """Few positions and a long axis: a launch of few workgroups, which is planned with cuts."""
    nt = 64
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=32, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=0,
             footprint_mode=0)
    H = random_table(np.random.default_rng(nz), nz, nt, 0)
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32", dtype)) as m:
        x = torch.randn(m.image_shape, device="cuda")
        ref = m.forward(x, dtype)
        exact = m.forward(x.double(), "fp64")
        assert float((ref - exact).norm() / exact.norm()) < (1e-2 if dtype == "bf16" else 1e-1)
        got = torch.full(m.signal_shape, 7.0, device="cuda")
        rc = _raw("aroam_forward_noalloc", m, dtype, x, got)
        torch.cuda.synchronize()
        if fits:
            assert rc == 0, P.aroam_last_error()
            assert torch.equal(got, ref)
        else:
            assert rc == -1 and "static buffer" in P.aroam_last_error()
            assert bool((got == 7.0).all())
