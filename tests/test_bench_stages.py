"""What the benchmark makes of the library's stage times."""
import os

import pytest

import bench
from launches import backward_call, launches
from path_cases import DY_ROWS, DY_TRANSPOSED

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


@pytest.fixture(scope="module")
def gathers(tmp_path_factory):
    """Matrices that the library's backward pass hands over transposed: the depth of that launch's grid (no such launch: 0)."""
    if not os.path.exists(bench.B.LIB_PATH):
        from paper_2403_07816_amd.build import build
        build(verbose=False)
    folder = str(tmp_path_factory.mktemp("launches"))
    return lambda *shape: sum(launch.grid[2] for rc, found in launches([backward_call(*shape, bench.B.BTX_BF16)], folder)
                              for launch in found if launch.kernel.startswith("gather_rows_t"))


@pytest.mark.parametrize("T,d,f,E,k,matrices", [
    (16384, 4096, 1376, 32, 8, 1), (16384, 4096, 11008, 4, 2, 2), (16384, 4096, 4096, 4, 2, 1), (16384, 4096, 4104, 4, 2, 2),
    (1 << 19, 4104, 1024, 4, 1, 2), *[(*c[:5], 1) for c in DY_ROWS], *[(*c[:5], 2) for c in DY_TRANSPOSED]])
def test_the_transposing_gather_is_charged_for_what_it_moves(gathers, T, d, f, E, k, matrices):
    """Read once and written once per routed slot: x, and dY too where dW2 does not read its token rows as they lie."""
    ran = bench.hbm_stages(dict(BACKWARD, gather_x_bwd=0.2), T, d, f, E, k)
    assert gathers(T, d, f, E, k) == matrices
    assert ran["gather_x_bwd"]["bytes_per_token"] == matrices * 2 * k * d * 2


@pytest.mark.parametrize("name", bench.VARIANTS)
def test_the_benchmark_s_workloads_are_charged_for_what_they_move(gathers, name):
    V = bench.VARIANTS[name]
    shape = V["T"], bench.D_MODEL, V["f"], V["E"], V["k"]
    assert bench.hbm_stages(dict(BACKWARD, gather_x_bwd=0.2), *shape)["gather_x_bwd"]["bytes_per_token"] == \
        gathers(*shape) * 2 * V["k"] * bench.D_MODEL * 2
