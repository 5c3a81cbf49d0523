"""The signal filter at the edges of its tiles: records shorter than a thread's outputs, one
sample past a workgroup's rows or samples, filters as long as the record, scans whose positions
do not fill the last workgroup.

Tolerance: an output is a sum of at most 2 L + 1 products; the roundings of its partial sums grow
like their square root times the unit roundoff and the sum of the absolute products (factor 2),
and 8 roundoffs cover the taps and single products."""
import numpy as np
import pytest

import workloads as W
from oracle import filters as ofil

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2009_10173_amd as P  # noqa: E402


@pytest.mark.parametrize("ny,nx,nt,L", [(1, 1, 3, 2), (1, 5, 8, 7), (2, 3, 9, 0), (3, 3, 31, 30),
                                        (5, 7, 64, 5), (1, 9, 65, 33), (3, 11, 257, 16),
                                        (1, 2, 2049, 100), (1, 3, 1023, 1000)])
def test_signal_filter_at_tile_edges(ny, nx, nt, L):
    cfg = W.config("tiny")
    g = W.grid(nx, 10e-6, 2, 10e-6, nt, 0, 0, ny=ny)
    f = dict(f_lo_hz=0.5e6, f_hi_hz=80e6, half_taps=L)
    h = ofil.bandpass_taps(f["f_lo_hz"], f["f_hi_hz"], g["fs_hz"], L)
    y = np.random.default_rng(nt + L).standard_normal((ny, nx, nt))
    with P.Model(cfg["sensor"], g, dtypes=("fp64", "fp32"), filter=f) as m:
        for npt, u in ((np.float64, 2.0 ** -53), (np.float32, 2.0 ** -24)):
            v = y.astype(npt)
            t = torch.empty(v.size + 1, dtype=torch.from_numpy(v).dtype, device="cuda")[1:]
            t = t.view(v.shape)
            t.copy_(torch.from_numpy(v))
            print(f"[filter {ny}x{nx} nt {nt} L {L} {npt.__name__}]", flush=True)
            got = m.filter_signals(t).cpu().numpy().astype(np.float64)
            ref = ofil.filter_time(v, h)
            bound = (2 * np.sqrt(2 * L + 1) + 8) * u * ofil.filter_time(np.abs(v), np.abs(h))
            assert np.all(np.abs(got - ref) <= bound)
