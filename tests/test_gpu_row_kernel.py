"""Particle-free boxes at the edges of the row rules: rows of 64 nodes whose
count per plane does not fill whole blocks of four run in tiles, and so do rows
past 512 nodes; in FP32 the other multiples of 64 are a tile each, bit for bit
as a batch's tiles of 64. Against the oracle at the gates of the parity tests."""
import numpy as np
import pytest

from paper_1109_3277_amd.workloads import System, uniform_fields
from tests.parity_util import check, compare, log, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tau,gate", [("fp64", 1.25, 1e-12), ("fp32", 1.0, 1e-5), ("fp16_dev", 1.0, 1e-3)])
@pytest.mark.parametrize("dims", [(64, 6, 5), (64, 7, 4), (64, 5, 9), (128, 5, 4), (192, 5, 7), (320, 4, 5), (384, 7, 4),
                                  (448, 4, 5), (576, 4, 4)])
def test_row_widths(dims, prec, tau, gate):
    ra, rb = uniform_fields(dims, sum(dims), 0.7, 0.7, 0.01)
    s = System(f"rows{dims}", dims, tau, 0.08, ra, rb)
    log(f"case {s.name} {prec}")
    o, g = run_oracle(s, 20), run_gpu(s, 20, prec)
    res = compare(o, g, s.dims, s.radii)
    log(f"  {res}")
    if prec == "fp16_dev":
        assert res["e_rho"] <= gate, res
    else:
        check(res, gate, particles=False)
    if dims[0] in (192, 320, 384, 448):
        from paper_1109_3277_amd.binding import Batch

        b = Batch([{"dims": dims, "tau": tau, "g_br": 0.08, "psi_kind": s.psi_kind}], prec)
        b[0].init_fields(ra, rb)
        b.step(20)
        assert all(np.array_equal(u, v) for u, v in zip(g.read_fields(), b[0].read_fields()))
        b.close()
    g.close()
