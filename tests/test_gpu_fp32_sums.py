"""FP32 applies are as close to 64 bits as sums of FP32 products are, for dense and sparse operands
alike, down to outputs of one product.

The yardstick adds an output's products one after another with one rounding each, as FP32 fused
multiply-adds do.  The kernel adds the products of a bundle (32 of them, in parts) apart from the
running sum, and leaves out products of parts below 2^-24 of theirs: 0.24 u rms (u = 2^-24),
against 0.58 u of a rounding.  One product: sqrt(0.58^2 + 0.24^2) / 0.58 = 1.08 of the yardstick's
error, held to 1.15.  Two products in two bundles, the worst of the short sums: two roundings and
left-out parts of the products and one rounding of their sum, against one and one: 1.20, held to
1.25.  A single product is off by no more than its rounding (u), the left-out ones (u) and 2^-5 u for
the sums of the smaller parts."""
import numpy as np
import pytest

from oracle import operators as oops
from test_gpu_apply_shapes import odd_start, on_scan, random_table

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402

U = 2.0 ** -24


def fma_sums(H, v, adjoint):
    """The apply as FP32 sums of one rounding per product (FP32 products are exact in FP64)."""
    K, (nz, nt) = (H.shape[0] - 1) // 2, H.shape[2:]
    ny, nx = v.shape[:2]
    out = np.zeros((ny, nx, nz if adjoint else nt), np.float32)
    big = np.pad(v.astype(np.float64), ((K, K), (K, K), (0, 0)))
    for dy in range(-K, K + 1):
        for dx in range(-K, K + 1):
            h = H[dy + K, dx + K] if not adjoint else H[dy + K, dx + K].T
            s = -1 if adjoint else 1
            w = big[K + s * dy:K + s * dy + ny, K + s * dx:K + s * dx + nx]
            for j in np.flatnonzero(h.any(1) & w.any((0, 1))):
                out = (out.astype(np.float64) + w[..., j, None] * h[j]).astype(np.float32)
    return out.astype(np.float64)


@pytest.mark.parametrize("op_name", ["forward", "adjoint"])
@pytest.mark.parametrize("density,most", [(1.0, 1.25), (0.1, 1.25), (0.01, 1.25), (0.003, 1.25),
                                          (0.0, 1.15)])
def test_fp32_applies_are_as_close_as_fp32_sums(density, most, op_name):
    K, nz, nt = 4, 33, 95
    ny, nx = (11, 35) if density else (2 * K + 1, 65 * (2 * K + 1))
    rng = np.random.default_rng(17)
    H = random_table(rng, nz, nt, K).astype(np.float32).astype(np.float64)
    op, n_in = getattr(oops, op_name), nz if op_name == "forward" else nt
    v = rng.standard_normal((ny, nx, n_in)).astype(np.float32)
    if density:
        v *= rng.random(v.shape) < density
    else:  # inputs so far apart that an output meets one of them
        one = np.zeros(v.shape, bool)
        cols = np.arange(K, nx, 2 * K + 1)
        one[K, cols, rng.integers(0, n_in, cols.size)] = True
        v *= one
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32")) as m:
        got = getattr(m, op_name)(odd_start(v, torch.float32), "fp32").cpu().numpy()
    ref = on_scan(op, H, v.astype(np.float64))
    yard = fma_sums(H, v, op_name == "adjoint")
    assert np.abs(yard - ref).max() < 1e-3
    mine, theirs = np.linalg.norm(got - ref), np.linalg.norm(yard - ref)
    print(f"[density {density:g} {op_name}: {mine / theirs:.3f} of the error of FP32 sums]", flush=True)
    assert mine <= most * theirs
    if not density:
        on = ref != 0
        assert not got[~on].any()
        worst = float((np.abs(got - ref)[on] / np.abs(ref[on])).max())
        print(f"[one product: worst error {worst / U:.3f} u]", flush=True)
        assert worst <= U * (2 + 2.0 ** -5)
