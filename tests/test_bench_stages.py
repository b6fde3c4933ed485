"""What the benchmark makes of the library's stage times."""
import pytest

import bench

FORWARD = dict(route=0.1, up_swiglu=2.0, down=1.0, combine=0.1)
BACKWARD = dict(FORWARD, bwd_act=1.0, bwd_dx=2.0, dw13=2.0, dw2=1.0, router_bwd=0.1)


@pytest.mark.parametrize("ran,dw13,dw2,total", [
    (FORWARD, None, None, 6), (dict(BACKWARD, gather_x_bwd=0.2), 4, 2, 18),
    # weight gradients from the rows as they lie: one launch, and an interval with nothing in it (or never recorded)
    (dict(BACKWARD, dw2=0.002), 6, None, 18), (dict(BACKWARD, dw2=0.0), 6, None, 18),
    (dict(BACKWARD, dw13=0.0, dw2=0.0), None, None, 12)])          # frozen experts
def test_products_are_charged_to_the_stage_that_does_them(ran, dw13, dw2, total):
    flops = bench.gemm_flops({name: ran.get(name, 0.0) for name in bench.B.STAGE_NAMES})
    assert (flops.get("dw13"), flops.get("dw2"), sum(flops.values())) == (dw13, dw2, total)
    assert all(ran[name] > 0 for name in flops)
