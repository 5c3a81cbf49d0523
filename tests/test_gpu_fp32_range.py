"""FP32 applies over the range of FP32: operands and table entries of any size.

The kernels split FP32 values into BF16 parts, so the cases are those in which a split could lose
bits: operands from subnormal to the largest, tables of one size or of entries far apart.

Tolerance: u = 2^-24 times (2 sqrt(n) + 8) times the sum of the n absolute products, as at the tile
edges, and for results near the smallest numbers n + 8 roundings to a multiple of 2^-149."""
import numpy as np
import pytest

from oracle import operators as oops
from test_gpu_apply_shapes import odd_start, on_scan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402

U = 2.0 ** -24
TINY = 2.0 ** -149


def grid_of(ny, nx, nz, nt, K):
    return dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt,
                k_half=K, footprint_mode=0)


def spread(rng, shape, low, high):
    """Values of either sign whose logarithms are uniform between 2^low and 2^high."""
    v = np.exp2(rng.uniform(low, high, shape)) * rng.choice((-1.0, 1.0), shape)
    return v.astype(np.float32).astype(np.float64)


# (table, operand): exponents between which the entries lie
RANGES = {
    "small operands": ((-2, 2), (-121, -117)),
    "subnormal operands": ((20, 24), (-146, -128)),
    "large operands": ((-22, -18), (124, 127.9)),
    "small table": ((-125, -121), (10, 14)),
    "small table, large operands": ((-125, -121), (100, 104)),
    "large table": ((118, 122), (-122, -110)),
    "operands far apart": ((-2, 2), (-140, 90)),
    "table far apart": ((-145, 60), (-2, 2)),
    "both far apart": ((-120, 20), (-100, 80)),
}


@pytest.mark.parametrize("name", RANGES)
@pytest.mark.parametrize("rows", [4, 8])
def test_fp32_applies_keep_fp32_precision_at_any_size(name, rows):
    """A sparse table (few products an output, so that small ones are alone in some)."""
    ny, nx, nz, nt, K = (9, 33, 17, 95, 4) if rows == 4 else (70, 130, 10, 600, 37)
    (ta, tb), (xa, xb) = RANGES[name]
    rng = np.random.default_rng(ny + len(name))
    H = np.zeros((2 * K + 1, 2 * K + 1, nz, nt))
    for i in range(3):
        dy, dx = (K, K) if i == 0 else rng.integers(0, 2 * K + 1, 2)
        on = rng.random((nz, nt)) < 0.2
        H[dy, dx][on] = spread(rng, int(on.sum()), ta, tb)
    with P.Model.from_table(grid_of(ny, nx, nz, nt, K), H, dtypes=("fp64", "fp32")) as m:
        for op_name in ("forward", "adjoint"):
            op, n_in = getattr(oops, op_name), nz if op_name == "forward" else nt
            v = spread(rng, (ny, nx, n_in), xa, xb) * (rng.random((ny, nx, n_in)) < 0.3)
            print(f"[{name}, {rows} rows, {op_name}]", flush=True)
            got = getattr(m, op_name)(odd_start(v.astype(np.float32), torch.float32), "fp32")
            got = got.cpu().numpy().astype(np.float64)
            ref = on_scan(op, H, v)
            size = on_scan(op, np.abs(H), np.abs(v))
            terms = on_scan(op, (H != 0).astype(np.float64), (v != 0).astype(np.float64))
            bound = (2 * np.sqrt(terms) + 8) * U * size + (terms + 8) * TINY
            sure = size * (1 + (terms + 8) * U) < np.finfo(np.float32).max
            assert sure.mean() > 0.5
            assert np.all(np.abs(got - ref)[sure] <= bound[sure])


def test_fp32_packs_hold_the_rounded_table_whatever_its_range():
    rng = np.random.default_rng(5)
    for low, high in ((-2, 2), (-125, -121), (118, 122), (-145, 60)):
        H = np.zeros((5, 5, 7, 40))
        on = rng.random(H.shape) < 0.3
        H[on] = np.exp2(rng.uniform(low, high, int(on.sum()))) * rng.choice((-1.0, 1.0), int(on.sum()))
        with P.Model.from_table(grid_of(6, 7, 7, 40, 2), H, dtypes=("fp64", "fp32")) as m:
            for adjoint in (False, True):
                got = m.export_quantized("fp32", adjoint)[0]
                assert np.array_equal(got, H.astype(np.float32).astype(np.float64)), (low, adjoint)
