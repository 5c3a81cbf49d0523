"""BF16 and FP8 applies at the edges of their tilings, against the oracle's operators on the
quantised table and operand: inner lengths around a run, a chunk and a scale chunk, scans around a
tile and a patch, the widest footprint (whose last units reach past the padded rows), vectors that
start at an odd element.

Tolerance: as for the FP32 applies a sum of n exact products errs by less than (2 sqrt(n) + 8) 2^-24
of the sum of the absolute products; the block-scaled FP8 MFMA adds up to 2^-13 of that sum
(tests/test_gpu_quantized.py)."""
import numpy as np
import pytest

from oracle import operators as oops
from oracle import quantize as Q
from tests.test_gpu_apply_shapes import odd_start, on_scan, random_table

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402

# (ny, nx, nz, nt, K)
GRIDS = [(1, 1, 1, 5, 0), (3, 17, 8, 31, 2), (4, 32, 33, 65, 2), (9, 33, 31, 130, 4),
         (13, 30, 96, 129, 6), (17, 20, 9, 150, 12), (3, 5, 9, 40, 97), (26, 70, 66, 257, 9)]


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_quantized_apply_matches_oracle_at_tile_edges(grid, dtype):
    ny, nx, nz, nt, K = grid
    rng = np.random.default_rng(1000 * ny + nx)
    if K > 20:  # columns at a few offsets, corners included
        H = np.zeros((2 * K + 1, 2 * K + 1, nz, nt))
        some = random_table(rng, nz, nt, 1)
        for i, (a, b) in enumerate([(K, K), (0, 0), (2 * K, 2 * K), (K + 2, K - 4), (K - 2, K + 3)]):
            H[a, b] = some[i // 3, i % 3]
    else:
        H = random_table(rng, nz, nt, K)
    Hq, lo, hi, _ = Q.quantize_table(H, dtype, delta=1e-11 * np.max(np.abs(H)))
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    with P.Model.from_table(g, H, dtypes=("fp64", dtype)) as m:
        for name in ("forward", "adjoint"):
            op, shape = getattr(oops, name), (ny, nx, nz if name == "forward" else nt)
            v = rng.standard_normal(shape).astype(np.float32)
            vq = Q.quantize_operand(v, "bf16" if dtype == "bf16" else "fp8-operand")
            print(f"[{grid} {dtype} {name}]", flush=True)
            got = getattr(m, name)(odd_start(v, torch.float32), dtype).cpu().numpy()
            ref = on_scan(op, Hq, vq.astype(np.float64))
            terms = on_scan(op, (H != 0).astype(np.float64), np.ones(shape)).max()
            mass = on_scan(op, np.abs(Hq), np.abs(vq).astype(np.float64))
            bound = (2 * np.sqrt(terms) + 8) * 2.0 ** -24 * mass
            if dtype == "fp8":
                bound = bound + 2.0 ** -13 * mass
            if np.any(hi != lo):
                bound = bound + on_scan(op, hi - lo, np.abs(vq).astype(np.float64))
            assert np.all(np.abs(got - ref) <= bound)
