"""Workspace sizes over the whole range of the particle capacity (host only)."""
import ctypes as C

import pytest

from paper_1109_3277_amd import binding as B


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_workspace_grows_by_a_fixed_amount_per_particle(prec):
    lib = B.load_library()

    def need(cap, batch=False):
        p = B.make_params((16, 16, 16), 1.0, 0.08, precision=prec, max_particles=cap, max_radius=1.0)
        return int(lib.lb_batch_workspace_bytes(1, C.byref(p)) if batch else lib.lb_workspace_bytes(C.byref(p)))

    per = (need(1 << 21) - need(1 << 20)) >> 20
    assert per > 0
    for cap in (1 << 22, 1 << 26, (1 << 27) - 1, 1 << 27, (1 << 28) + 5, 1 << 30, (1 << 31) - 1):
        # every buffer is rounded up to 256 bytes, some 20 of them
        assert abs(need(cap) - need(1 << 20) - (cap - (1 << 20)) * per) <= 20 * 256, cap
        assert need(cap, batch=True) > need(cap), cap
