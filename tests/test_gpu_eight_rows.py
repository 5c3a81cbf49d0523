"""FP32 applies on patches of eight rows (K from 35 to 40, launches that fill the chip), where the
length of the inner axis is no multiple of the vectors that are staged and where it is, and the
position tiles end inside a patch.

Tables and tolerance: as for the wide footprints at the tile edges."""
import numpy as np
import pytest

from oracle import operators as oops
from test_gpu_apply_shapes import odd_start, on_scan, random_table
from test_launch_plan_costs import ring_rows  # noqa: F401  (fixture: the rule, built on the host)

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402

CUS = 256
# (ny, nx, nz, nt, K, operator): output tiles x patches at least 1.5 times the rule's threshold
CASES = [(70, 130, 9, 600, 35, "forward"), (69, 97, 8, 1000, 40, "forward"),
         (61, 113, 27, 900, 37, "forward"), (100, 160, 480, 21, 36, "adjoint"),
         (97, 146, 500, 20, 40, "adjoint")]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_the_cases_are_taken_by_eight_rows(case, ring_rows):  # noqa: F811
    ny, nx, nz, nt, K, name = case
    tiles = -(-(nt if name == "forward" else nz) // 16)
    assert ring_rows(K, tiles, nx, ny, CUS) == 8
    assert ring_rows(K, tiles, nx, ny, CUS * 3 // 2) == 8


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_eight_row_applies_match_oracle(case):
    ny, nx, nz, nt, K, name = case
    assert torch.cuda.get_device_properties(0).multi_processor_count == CUS
    rng = np.random.default_rng(nt)
    full = random_table(rng, nz, nt, 2)
    H = np.zeros((2 * K + 1, 2 * K + 1, nz, nt))
    for i, (a, b) in enumerate([(K, K), (0, 0), (2 * K, 0), (0, 2 * K), (2 * K, 2 * K)]):
        H[a, b] = full[i, 0]
    for i in range(30):
        H[rng.integers(0, 2 * K + 1), rng.integers(0, 2 * K + 1)] = full[i % 5, 1 + i % 4]
    op, shape = getattr(oops, name), (ny, nx, nz if name == "forward" else nt)
    v = rng.standard_normal(shape).astype(np.float32)
    g = dict(c_mps=1500.0, fs_hz=250e6, nx=nx, ny=ny, step_m=1e-5, nz=nz, dz_m=1e-5, nt=nt, k_half=K,
             footprint_mode=0)
    with P.Model.from_table(g, H, dtypes=("fp64", "fp32")) as m:
        print(f"[eight rows {case}]", flush=True)
        got = getattr(m, name)(odd_start(v, torch.float32), "fp32").cpu().numpy().astype(np.float64)
    ref = on_scan(op, H, v.astype(np.float64))
    terms = on_scan(op, (H != 0).astype(np.float64), np.ones(shape)).max()
    bound = (2 * np.sqrt(terms) + 8) * 2.0 ** -24 * on_scan(op, np.abs(H), np.abs(v).astype(np.float64))
    assert np.all(np.abs(got - ref) <= bound)
