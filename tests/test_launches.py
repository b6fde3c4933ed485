"""What the library launches for given sizes, without a GPU (see launches.py)."""
import math
import os
import re

import pytest

from paper_2403_07816_amd import binding as B

from launches import P, adamw_call, backward_call, forward_call, host_seconds, launches, route_call
from path_cases import (ANY, BWD_ACT, BWD_DX, DOWN, DY_ROWS, DY_TRANSPOSED, F32_LAST_ROUND, FEW_K_TILES, HALF, JOINT_FORWARD, LAST_ROUND_CUT, ROUTE_AHEAD, ROUTE_MANY, ROW_PITCH,
                        TILED_FORWARD, TRANSPOSED_ROWS, UP, WHOLE, WHOLE_TILE_CASES, whole_tile_case)

MAX_THREADS = (1 << 32) - 1     # of one launch and direction of the grid


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if not os.path.exists(B.LIB_PATH):
        from paper_2403_07816_amd.build import build
        build(verbose=False)
    folder = tmp_path_factory.mktemp("launches")
    return lambda *calls: launches(list(calls), str(folder))


def threads_fit(launch):
    return all(g * b <= MAX_THREADS for g, b in zip(launch.grid, launch.block))


@pytest.mark.parametrize("dtype", [B.BTX_F32, B.BTX_BF16])
@pytest.mark.parametrize("n", [1, 4097, (1 << 34) - 1024, (1 << 34) + 5, 1 << 36])
def test_adamw_takes_tensors_of_any_length(record, n, dtype):
    """Every element belongs to one launch, in pieces of whole 16-byte chunks where one launch cannot hold the threads."""
    (rc, found), = record(adamw_call(n, dtype))
    assert rc == 0 and found
    done = 0
    for launch in found:
        assert threads_fit(launch)
        assert launch.first == P + 4 * done and done % 4 == 0       # the master weights of this piece
        done += launch.grid[0] * 1024                               # at most; the last workgroup may hold fewer
    assert done - 1024 < n <= done + 3                              # (up to 3 trailing elements go to the first workgroup)


def test_a_workspace_for_many_tokens_serves_fewer(record):
    """Programs size their workspace for the largest batch: no query may fall as the number of tokens grows."""
    shapes = [(512, 1376, 8, 2), (64, 2056, 3, 2), (4096, 688, 64, 8), (2048, 5504, 8, 2), (72, 96, 4, 1), (1032, 264, 64, 4)]
    tokens = sorted({1, 2, 3, 17, 40, 64, 100, 255, 256, 440, 700, 768, 769, 880, 881, 882, 1000, 1345, 1500, 2003, 2304, 2305, 2561,
                     3000, 4001, 4096, 16384, *range(216, 232), *range(840, 884)})
    calls = [(f"btx_moe_ff_{which}_workspace_bytes", [T, d, f, E, k, dtype])
             for which in ("forward", "backward") for d, f, E, k in shapes for dtype in (B.BTX_F32, B.BTX_BF16) for T in tokens]
    sizes = [rc for rc, _ in record(*calls)]
    for (name, args), size, (next_name, next_args), next_size in zip(calls, sizes, calls[1:], sizes[1:]):
        if name == next_name and args[1:] == next_args[1:]:
            assert size <= next_size, f"{name}: {args} {size} bytes, {next_args} {next_size}"


@pytest.mark.parametrize("T,d,f,E,k,forward_kb,backward_kb", [(1, 1032, 264, 64, 4, 64, 22000), (16, 264, 200, 4, 2, 64, 700),
                                                              (70, 8, 8, 2, 1, 64, 64), (301, 520, 392, 4, 2, 3000, 6000)])
def test_bf16_workspaces_of_small_layers_are_small(record, T, d, f, E, k, forward_kb, backward_kb):
    """The sums of K slices take what these products can need, not the 84 MB of the largest ones."""
    (forward, _), (backward, _) = record(*((f"btx_moe_ff_{which}_workspace_bytes", [T, d, f, E, k, B.BTX_BF16])
                                           for which in ("forward", "backward")))
    assert 0 < forward <= forward_kb << 10
    assert 0 < backward <= backward_kb << 10


@pytest.mark.parametrize("T,d,f,E,k,transposed", [
    (16384, 4096, 1376, 32, 8, 1), (16384, 4096, 4096, 4, 2, 1), (16384, 4096, 4104, 4, 2, 2), (1 << 19, 4104, 1024, 4, 1, 2)])
def test_bf16_workspaces_hold_the_matrices_that_are_transposed(record, T, d, f, E, k, transposed):
    """x, ga and dY, but no dY where dW2 reads its token rows; and dxs, dh1, dh3, partial sums of d gates, rows that are gathered."""
    (size, _), = record(("btx_moe_ff_backward_workspace_bytes", [T, d, f, E, k, B.BTX_BF16]))
    R, pitch = T * k, T * k + 64 * E
    gathered = R * d if T * d * 2 >= 1 << 32 else 0
    least = 2 * (transposed * d * pitch + f * pitch + R * d + 2 * R * f + gathered)
    assert least <= size < least + d * pitch            # half of a matrix more at most


@pytest.mark.parametrize("T,d,f,E,k", [case[:5] for case in ROW_PITCH])
def test_bf16_workspaces_hold_rows_that_start_on_whole_lines(record, T, d, f, E, k):
    """From 136 to 65536 columns; ga has room for either order, transposed rows of an expert starting at multiples of 64."""
    (forward, _), (backward, _) = record(*((f"btx_moe_ff_{which}_workspace_bytes", [T, d, f, E, k, B.BTX_BF16]) for which in ("forward", "backward")))
    R, columns = T * k, math.ceil(f / 64) * 64 if 128 < f <= 65536 else f
    ga = max(R * columns, (math.ceil(R / 64) * 64 + 64 * E) * f)
    assert forward >= 2 * R * (columns + d) and backward >= 2 * (2 * R * columns + ga + 2 * R * d)


@pytest.mark.parametrize("dW_dtype", [B.BTX_F32, B.BTX_BF16])
def test_strips_of_weight_gradients_are_streamed_from_half_lines_on(record, dW_dtype):
    """The strips' stores go past the caches where every row starts on 64 bytes: not for a stack that starts on any other 16-byte
    piece, nor with an expert stride that shifts the others there."""
    def streamed(T, dW2=P, stride=None, d=256, f=192):
        (rc, found), = record(backward_call(T, d, f, 8, 2, B.BTX_BF16, dW_dtype=dW_dtype, dW2=dW2, stride=stride))
        last = [n.kernel for n in found if "dw_strip" in n.kernel or ", 5, 0, " in n.kernel][-1]
        assert rc == 0 and ("strip" in last) == (T == 100)
        return last.endswith("true>")
    assert streamed(100) and streamed(100, dW2=P + 64) and streamed(100, stride=256 * 192 + 32)
    assert not streamed(100, dW2=P + 16) and not streamed(100, stride=256 * 192 + 8)
    wide = dict(d=2048, f=5504)                                    # 256 x 256 tiles: from anywhere
    assert streamed(1500, **wide) and streamed(1500, dW2=P + 16, **wide)


@pytest.mark.parametrize("T,d,f,E,k,direct", [
    (1, 64, 64, 64, 8, True), (720, 512, 5504, 4, 2, True), (722, 512, 5504, 4, 2, False), (722, 504, 520, 4, 2, True),
    (1250, 520, 1040, 2, 2, True), (1251, 520, 1040, 2, 2, False),
    # few strips: 700 rows of fewer than 512 columns, 2500 of more; from d x E = 4096 on any number of rows; 700 thousand below 512 columns
    (1500, 256, 192, 8, 2, True), (1400, 504, 520, 4, 2, True), (1402, 504, 520, 4, 2, False), (5000, 512, 352, 4, 2, True), (5002, 512, 352, 4, 2, False),
    (20000, 504, 64, 8, 2, False), (20000, 512, 64, 8, 2, True), (160000, 64, 64, 64, 2, True), (6000, 504, 1400, 24, 2, True), (6012, 504, 1400, 24, 2, False)])
def test_weight_gradients_of_few_rows_read_token_rows(record, T, d, f, E, k, direct):
    """Up to 360 rows per expert, or rows x width of 1.3 million where there are strips enough, nothing is transposed for the weight
    gradients."""
    (rc, found), = record(backward_call(T, d, f, E, k, B.BTX_BF16))
    names = " ".join(launch.kernel for launch in found)
    assert rc == 0 and ("dw_strip" in names) == direct and ("gather_rows_t" in names) == (not direct)


@pytest.mark.parametrize("T,d,f,E,k,direct", [(720, 512, 5504, 4, 2, True), (10000, 512, 64, 8, 2, True), (10004, 512, 64, 8, 2, False), (20000, 1024, 64, 8, 2, True)])
def test_fp32_weight_gradients_of_few_strips_transpose_earlier(record, T, d, f, E, k, direct):
    (rc, found), = record(backward_call(T, d, f, E, k, B.BTX_BF16, dW_dtype=B.BTX_F32))
    assert rc == 0 and any("gather_rows_t" in launch.kernel for launch in found) == (not direct)


@pytest.mark.parametrize("case", TRANSPOSED_ROWS)
def test_shapes_of_transposed_rows_take_that_path(record, case):
    (rc, found), = record(backward_call(*case[:5], B.BTX_BF16))
    assert rc == 0 and any("gather_rows_t" in launch.kernel for launch in found)


@pytest.mark.parametrize("case,rows", [(c, True) for c in DY_ROWS] + [(c, False) for c in DY_TRANSPOSED] +
                         [((16384, 4096, 4096, 4, 2), True), ((16384, 4096, 4104, 4, 2), False), ((1 << 19, 4104, 1024, 4, 1), False), ((500_000, 4104, 72, 1, 1), True),
                          ((16384, 4096, 1376, 1, 1), True), ((16384, 4088, 1376, 1, 1), False), ((16384, 256, 4096, 16, 2), True), ((16384, 248, 4096, 17, 2), False),
                          ((16384, 520, 2768, 8, 2), True), ((16384, 520, 2776, 8, 2), False), ((16384, 64, 1376, 64, 8), False)])
def test_dW2_of_tiles_reads_token_rows_of_dY(record, case, rows):
    """Experts of up to 4096 columns, counted as the tiles' columns of d go over its own, and d times experts from 4096 on, unless the
    rows' offsets need more than 32 bits; x alone is transposed then."""
    (rc, found), = record(backward_call(*case[:5], B.BTX_BF16))
    gather, = [launch for launch in found if launch.kernel.startswith("gather_rows_t")]
    dw2, = [launch for launch in found if ", 5, 0, " in launch.kernel]
    assert rc == 0 and gather.grid[2] == (1 if rows else 2) and dw2.kernel.startswith("mfma_gemm_kernel_rows") == rows


@pytest.mark.parametrize("dtype,T,d,E,beside", [(B.BTX_BF16, 64, 256, 4, True), (B.BTX_BF16, 1792, 1024, 16, True), (B.BTX_BF16, 1793, 1024, 16, False),
                                                (B.BTX_F32, 4864, 2048, 8, True), (B.BTX_F32, 4865, 2048, 8, False)])
def test_router_gradient_beside_the_weight_gradients(record, dtype, T, d, E, beside):
    """As long as its workgroups (4 tokens, or 256 weights of the router) are no more than run at a time: 512, fp32 1280."""
    (rc, found), = record(backward_call(T, d, 64, E, 2, dtype))
    assert rc == 0 and any("router_ds_kernel" in launch.kernel for launch in found) != beside


@pytest.mark.parametrize("dtype", [B.BTX_F32, B.BTX_BF16])
@pytest.mark.parametrize("T,d,E,beside", [(64, 64, 1, True), (16320, 4096, 4, True), (16321, 4096, 4, False), (32704, 2048, 8, True), (32705, 2048, 8, False)])
def test_large_batches_finish_dX_in_a_kernel_of_its_own(record, dtype, T, d, E, beside):
    """512 blocks of 64 tokens and 2048 columns: nothing runs beside dX, and its kernel holds nothing for that."""
    (rc, found), = record(backward_call(T, d, 64, E, 1, dtype))
    names = " ".join(launch.kernel for launch in found)
    assert rc == 0 and ("dx_and_dwr_kernel" in names) == beside
    assert ("dx_finish_kernel" in names and "dwr_partial_kernel" in names) == (not beside)


@pytest.mark.parametrize("dtype,T,d,E,beside", [
    (B.BTX_BF16, 1501, 4096, 64, True), (B.BTX_F32, 609, 4096, 33, True), (B.BTX_BF16, 3122, 3072, 64, True), (B.BTX_BF16, 13616, 1032, 24, True),
    # 84 MB of fp32 rows that are read again, 144 MB of bf16 ones
    (B.BTX_F32, 2563, 2048, 64, True), (B.BTX_F32, 2564, 2048, 64, False), (B.BTX_BF16, 4394, 4096, 64, True), (B.BTX_BF16, 4395, 4096, 64, False),
    # dX's last round of workgroups nearly full, more than 1536 workgroups together
    (B.BTX_BF16, 15872, 256, 64, True), (B.BTX_BF16, 5400, 1032, 64, False), (B.BTX_BF16, 8000, 1544, 17, False), (B.BTX_BF16, 7136, 1544, 17, True)])
def test_partial_sums_of_many_experts_router_gradient_beside_dX(record, dtype, T, d, E, beside):
    (rc, found), = record(backward_call(T, d, 64, E, 2, dtype))
    names = " ".join(launch.kernel for launch in found)
    assert rc == 0 and ("dx_and_dwr_lds" in names) == beside and ("dwr_partial_few" in names and "dx_finish_lds" in names) == (not beside)


@pytest.mark.parametrize("f,launches", [(1_000_000, 1), (8_000_000, 4)])
def test_fp32_backward_products_that_fit_no_launch_together(record, f, launches):
    """Each of them fits: the router's gradient, dX, dW1 and dW3, dW2."""
    (rc, found), = record(backward_call(64, 8, f, 64, 2, B.BTX_F32))
    assert rc == 0 and all(threads_fit(launch) for launch in found)
    assert sum(launch.kernel.startswith(("f32_dx_dw", "f32_gemm_kernel<3", "f32_gemm_kernel<4", "f32_gemm_kernel<5")) for launch in found) == launches


@pytest.mark.parametrize("T,d,f,E,k,stages", [
    (37, 3984, 216, 16, 2, 3), (4, 3896, 816, 64, 2, 3), (1, 680, 8192, 2, 2, 3),
    # W1 and W3 of less than 88 MB; more than 512 tiles; tokens of fewer experts
    (1, 664, 8192, 2, 2, 2), (512, 512, 1376, 8, 2, 2), (1, 680, 8224, 2, 2, 2), (443, 3824, 1488, 8, 2, 2), (1, 3896, 816, 64, 2, 2)])
def test_fp32_up_projection_of_weights_from_memory_has_three_stages(record, T, d, f, E, k, stages):
    (rc, found), = record(forward_call(T, d, f, E, k, B.BTX_F32))
    up, = [launch.kernel for launch in found if launch.kernel.startswith("f32_gemm_kernel<0")]
    assert rc == 0 and up.endswith(f", {stages}>")


@pytest.mark.parametrize("T,E,k", [(4_000_000, 2, 1), (2_000_000, 2, 2), (1_500_000, 8, 2), (4_000_000, 1, 1)])
def test_many_fp32_rows_cost_the_host_no_more_than_few(tmp_path, T, E, k):
    """The expected tiles of DOWN's last round are counted without a step for each of them (117 us beside 5 at 2 000 000 rows of an expert)."""
    few, many = (host_seconds(forward_call(n, 256, 1376, E, k, B.BTX_F32, save=False), str(tmp_path)) for n in (5000, T))
    assert many < 5 * few + 50e-6


@pytest.mark.parametrize("case,cut", [(c, True) for c in F32_LAST_ROUND] + [
    # one tile more than others of a unit's, none, too many for two slices; few k tiles; fewer tiles than units
    ((2003, 512, 1376, 8, 2), True), ((1900, 512, 1376, 8, 2), False), ((2003, 512, 416, 8, 2), False), ((64, 512, 1376, 8, 2), False)])
def test_last_round_of_fp32_down_projections_is_cut(record, case, cut):
    T, d, f, E, k = case[:5]
    (size, _), (rc, found) = record(("btx_moe_ff_forward_workspace_bytes", [T, d, f, E, k, B.BTX_F32]), forward_call(T, d, f, E, k, B.BTX_F32))
    names = [launch.kernel for launch in found]
    assert rc == 0 and ("f32_cut_finish_kernel" in names) == cut
    if cut:
        down = found[names.index("f32_cut_finish_kernel") - 1]
        tiles = (math.ceil(T * k / 64) + E) * math.ceil(d / 64)    # at most; of each XCD's, 32 workgroups more
        assert down.kernel.startswith("f32_gemm_kernel<1") and down.grid[0] // 8 >= math.ceil(tiles / 8) + 32
        assert size >= 4 * (T * k * (f + d) + 256 * 64 * 64)       # act, y, and a tile's sums for every workgroup that has a slice


@pytest.mark.parametrize("T,d,f,E,k", [case[:5] for case in JOINT_FORWARD])
@pytest.mark.parametrize("save", [False, True])
def test_small_fp32_layers_forward_in_one_launch(record, T, d, f, E, k, save):
    (rc, found), = record(forward_call(T, d, f, E, k, B.BTX_F32, save=save))
    assert rc == 0 and [launch.kernel.split("<")[0] for launch in found] == ["f32_ff_kernel", "combine_kernel"]
    tiles = math.ceil(T * k / 16) + E                              # at most, of which 64 columns of f each
    assert tiles * math.ceil(f / 64) <= found[0].grid[0] < tiles * math.ceil(f / 64) + 8 and found[1].kernel.endswith("true>") == (f > 64)


@pytest.mark.parametrize("T,d,f,E,k,joint", [
    (1274, 192, 192, 2, 1, True), (1275, 192, 192, 2, 1, False), (16, 200, 64, 2, 2, False),      # 47 million products, 192 columns
    (16, 64, 2048, 2, 2, True), (16, 64, 2056, 2, 2, False), (16, 64, 512, 8, 8, True), (16, 64, 520, 8, 8, False), (16, 64, 64, 9, 9, True), (16, 64, 72, 9, 9, False),
    (100, 192, 256, 2, 1, True), (100, 192, 320, 2, 1, True), (100, 184, 176, 4, 2, True)])       # 64 slices over a token's slots; room for the sums
def test_limits_of_small_fp32_layers(record, T, d, f, E, k, joint):
    (rc, found), = record(forward_call(T, d, f, E, k, B.BTX_F32))
    assert rc == 0 and found[0].kernel.startswith("f32_ff_kernel" if joint else "f32_gemm_kernel<0")


@pytest.mark.parametrize("case,cut", TILED_FORWARD)
def test_fp32_forward_of_narrow_rows_takes_two_launches(record, case, cut):
    T, d, f, E, k, _ = case
    (rc, found), = record(forward_call(T, d, f, E, k, B.BTX_F32, save=False))
    up, down, *finish, combine = [launch.kernel for launch in found]
    assert rc == 0 and up.startswith("f32_gemm_kernel<0") and down.startswith("f32_gemm_kernel<1")
    # the slices' sums, which the combine adds for up to 8 slots
    assert finish == (["f32_slices_finish_kernel"] if cut and k > 8 else []) and combine.endswith("true>") == (cut and k <= 8)


@pytest.mark.parametrize("T,d,f,E,k,joint", [
    # many narrow rows: more workgroups than run at once; experts of fewer columns than a workgroup takes
    (16000, 8, 8, 1, 1, True), (16001, 8, 8, 1, 1, False), (4000, 8, 72, 2, 2, True), (4001, 8, 72, 2, 2, False), (300000, 16, 8, 4, 1, False),
    (11474, 64, 8, 1, 1, True), (11475, 64, 8, 1, 1, False), (13020, 192, 8, 1, 1, False), (1, 8, 4096, 1, 1, True)])
def test_rows_of_small_fp32_layers(record, T, d, f, E, k, joint):
    (rc, found), = record(forward_call(T, d, f, E, k, B.BTX_F32))
    assert rc == 0 and found[0].kernel.startswith("f32_ff_kernel" if joint else "f32_gemm_kernel<0")


def test_sums_of_small_fp32_layers_fit_the_workspace(record):
    """Their slices, [slice][T k, d] from the workspace's start on, at every number of columns: no more than the query asks for."""
    shapes = [(T, d, f, k) for T in (1, 33, 200) for k in (1, 2, 8) for d in range(8, 200, 8) for f in (8, 64, 72, 136, 256, 264, 520, 1024, 1376, 2048)]
    found = record(*(call for T, d, f, k in shapes for call in
                     (("btx_moe_ff_forward_workspace_bytes", [T, d, f, 8, k, B.BTX_F32]), forward_call(T, d, f, 8, k, B.BTX_F32))))
    taken = 0
    for (T, d, f, k), (size, _), (rc, launched) in zip(shapes, found[::2], found[1::2]):
        assert rc == 0
        if launched[0].kernel.startswith("f32_ff_kernel"):
            taken += 1
            assert math.ceil(f / 64) * T * k * d * 4 <= size, (T, d, f, k)
    assert taken > len(shapes) // 2


def test_fp32_products_of_too_many_tiles_are_refused(record):
    """2^24 tiles of 256 threads are more than a launch can hold (137 GB of activations)."""
    (rc, found), = record(forward_call(4_000_000, 64, 8704, 4, 1, B.BTX_F32, save=False))
    assert rc == 2 and not found
    (rc, found), = record(forward_call(4_000_000, 64, 8448, 4, 1, B.BTX_F32, save=False))
    assert rc == 0 and found and all(threads_fit(launch) for launch in found)


@pytest.mark.parametrize("n", [1, 1 << 20, (1 << 34) + 5])
def test_merges_of_any_length_fit_a_launch(record, n):
    """The kernels walk over the grid, so fewer threads than chunks are fine."""
    for name, args in (("btx_merge_average", [[P, P], 2, P, n, B.BTX_F32, 0]),
                       ("btx_merge_average", [[P, P], 2, P, n, B.BTX_BF16, 0]),
                       ("btx_merge_weighted", [[P, P], [0.5, 0.5], 2, P, n, B.BTX_F32, 0]),
                       ("btx_merge_weighted", [[P, P], [0.5, 0.5], 2, P, n, B.BTX_BF16, 0])):
        (rc, found), = record((name, args))
        assert rc == 0 and len(found) == 1 and threads_fit(found[0])


def bf16_products(record, T, d, f, E, k):
    """{product: (rows of a tile, form of the last k tile, a last round of it can be cut)} of a forward and a backward pass."""
    paths = {}
    for rc, found in record(forward_call(T, d, f, E, k, B.BTX_BF16), backward_call(T, d, f, E, k, B.BTX_BF16)):
        assert rc == 0
        names = [launch.kernel for launch in found]
        for name, following in zip(names, names[1:] + [""]):
            numbers = [int(n) for n in re.findall(r"[<,] ?(\d+)(?=[,>])", name)]
            if name.startswith("mfma_gemm_kernel"):
                paths[numbers[7]] = numbers[0], numbers[8], following.startswith("mfma_split_finish")
            elif name.startswith("mfma_small_kernel"):
                paths[numbers[5]] = numbers[0], numbers[6], False
    return paths


def slices_of_last_round(rows, E, N, K, product, tile):
    """Gemm::split_plan for `rows` rows on each of E experts and 256 compute units."""
    tiles = E * math.ceil(rows / tile) * math.ceil(N / (128 if product == UP else 256))
    left, k_tiles = tiles % 256, math.ceil(K / 64) * (2 if product == BWD_DX else 1)
    return max(1, min(8, 256 // left, k_tiles // 16)) if left else 1


@pytest.mark.parametrize("T,d,f,wide", [
    # 255 rows of K elements and 64 of their own, and at most 3 KB by which copies share a base: 2^32 bytes
    (257, 264, 8421496, ()), (257, 264, 8421504, (DOWN, BWD_DX)), (16, 8421504, 64, (UP, BWD_ACT)),
    # 64 rows of W1 and W3, or of W2
    (100, 8, (1 << 25) - 24, (DOWN, BWD_DX)), (100, 8, (1 << 25) - 16, (UP, DOWN, BWD_DX)), (8, (1 << 25) - 16, 8, (UP, DOWN, BWD_ACT))])
def test_bf16_operands_of_far_rows_take_64_bit_offsets(record, T, d, f, wide):
    taken = bf16_products(record, T, d, f, 1, 1)
    for product, (tile, tail, _) in taken.items():
        assert (tail == 3) == (product in wide) and (tile == 64 or tail != 3)
        if tail != 3:
            K = d if product in (UP, BWD_ACT) else f
            N = f + d - K if product in (UP, DOWN) else 0
            assert max((min(tile, T) - 1) * K + min(K, 64), min(64, K) * N) * 2 + 3072 <= 1 << 32


@pytest.mark.parametrize("T,f,status", [(400, (1 << 25) - 24, 0), (400, (1 << 25) - 16, 2), (100, 1 << 26, 0), (100, (1 << 26) + 8, 2), (20, 1 << 26, 0)])
def test_bf16_weight_gradients_of_rows_too_far_apart_are_refused(record, T, f, status):
    """64 grouped rows of the products' operands (strips: 32) span up to 2^32 bytes; without weight gradients any width will do."""
    name, args = backward_call(T, 8, f, 1, 1, B.BTX_BF16)
    frozen = list(args)
    frozen[-7:-4] = [0, 0, 0]
    (rc, found), (frozen_rc, frozen_found) = record((name, args), (name, frozen))
    assert rc == status and bool(found) == (status == 0)
    assert frozen_rc == 0 and frozen_found


@pytest.mark.parametrize("case,paths", LAST_ROUND_CUT)
def test_shapes_of_the_cut_last_round_take_that_path(record, case, paths):
    T, d, f, E, k, options = case
    taken = bf16_products(record, T, d, f, E, k)
    rows = math.ceil(T * k / E)
    if options.get("cf"):
        rows = min(rows, math.ceil(options["cf"] * T * k / E))
    for product, (tile, tail, slices) in paths.items():
        N, K = (f, d) if product == UP else (d, f)
        assert taken[product] == (tile, tail, True)
        # 192-row tiles know no HALF: a last k tile of 32 takes the general form there
        assert tail == (WHOLE if K % 64 == 0 else HALF if K % 64 == 32 and tile == 256 else ANY)
        assert slices_of_last_round(rows, E, N, K, product, tile) == slices > 1


@pytest.mark.parametrize("case", range(WHOLE_TILE_CASES))
def test_random_shapes_of_whole_tiles_take_that_path(record, case):
    T, d, f, E, k = whole_tile_case(case)
    taken = bf16_products(record, T, d, f, E, k)
    assert all(taken[product][0] == 256 for product in (UP, DOWN, BWD_ACT, BWD_DX)) and taken[BWD_DX][2]


@pytest.mark.parametrize("case,products", FEW_K_TILES)
def test_shapes_of_few_k_tiles_take_large_row_tiles(record, case, products):
    T, d, f, E, k, _ = case
    taken = bf16_products(record, T, d, f, E, k)
    assert all(taken[product][0] == 256 for product in products)


@pytest.mark.parametrize("dtype,T,d,threads", [(B.BTX_BF16, 8000, 8192, 1024), (B.BTX_BF16, 8192, 8192, 256), (B.BTX_F32, 4096, 8192, 1024),
                                               (B.BTX_F32, 4097, 8192, 256), (B.BTX_F32, 4097, 1024, 1024), (B.BTX_BF16, 100, 16384, 256)])
def test_normalisation_backward_groups_threads_where_that_is_faster(record, dtype, T, d, threads):
    (rc, found), = record(("btx_rmsnorm_backward", [P, P, P, P, P, dtype, T, d, P, P, P, 1 << 62, 0]))
    assert rc == 0 and found[0].block[0] == threads


@pytest.mark.parametrize("dtype,norm,T,d,E,waves", [
    # one workgroup of 16 tokens on a compute unit
    (B.BTX_BF16, False, 4096, 8192, 8, 8), (B.BTX_F32, False, 4096, 8200, 8, 4), (B.BTX_BF16, True, 4096, 4096, 4, 16),
    (B.BTX_BF16, True, 4096, 4096, 8, 8), (B.BTX_BF16, True, 4096, 1024, 64, 16), (B.BTX_F32, True, 4096, 512, 64, 16),
    (B.BTX_F32, True, 4096, 4096, 64, 8), (B.BTX_F32, True, 600, 16384, 64, 4),
    # two
    (B.BTX_BF16, False, 4097, 4096, 8, 4), (B.BTX_F32, False, 4097, 4096, 8, 8), (B.BTX_F32, False, 4097, 4096, 16, None),
    (B.BTX_BF16, True, 8176, 16384, 64, 8), (B.BTX_F32, True, 8176, 4096, 64, 4), (B.BTX_F32, True, 8176, 512, 64, 8),
    (B.BTX_BF16, True, 8177, 4096, 4, 4),
    # logits on the matrix cores: 8 wavefronts and one block of tokens, or 4 and two
    (B.BTX_BF16, False, 4096, 4096, 64, 8), (B.BTX_BF16, False, 4097, 512, 64, 4), (B.BTX_BF16, False, 4097, 2048, 32, 8),
    (B.BTX_BF16, False, 4097, 4096, 32, 4)])
def test_wavefronts_that_share_16_tokens(record, dtype, norm, T, d, E, waves):
    k = min(E, 2)
    lead = [P, dtype, P, 1e-5, 2 * P, P] if norm else [P, dtype]
    args = lead + [P, 0, 0, T, d, E, k, 0, 0, 0.01, 1.0, 0.0] + [P] * 10 + [P, 1 << 62, 0]
    (rc, found), = record(("btx_moe_norm_route" if norm else "btx_moe_route", args))
    tokens, = [launch for launch in found if launch.kernel.startswith("route_tokens")]
    assert rc == 0
    if waves is None:           # fp32 rows, 16 experts: the matrix cores
        assert "0, false, 8, 1, 1>" in tokens.kernel
    else:
        assert tokens.block[0] == 64 * waves and f", {waves}, " in tokens.kernel


@pytest.mark.parametrize("T,d,E,k,dtype", ROUTE_AHEAD)
def test_shapes_of_few_wide_rows_are_requested_ahead(record, T, d, E, k, dtype):
    (rc, found), = record(route_call(T, d, E, k, dtype, norm=True))
    assert rc == 0 and found[0].kernel.startswith("route_small_tokens") and found[0].kernel.endswith(", 2>")


@pytest.mark.parametrize("dtype,T,d,E,norm,ahead", [
    *[(B.BTX_BF16, *c) for c in [
        (16, 4096, 4, True, 2), (16, 2056, 16, True, 2), (256, 6144, 4, True, 2), (256, 6152, 4, True, 0), (512, 4096, 5, True, 2), (257, 4096, 4, True, 0),
        (16, 2048, 4, True, 0), (16, 4096, 17, True, 0), (16, 4096, 4, False, 0), (512, 8192, 8, True, 2), (16, 8200, 8, True, 0), (16, 8192, 16, True, 2),
        (16, 4096, 9, True, 0), (256, 3072, 12, True, 0)]],
    *[(B.BTX_F32, *c) for c in [(512, 4096, 4, True, 2), (512, 4096, 8, True, 2), (16, 4104, 4, True, 0), (16, 2048, 4, True, 0), (16, 4096, 9, True, 0), (16, 4096, 16, True, 0)]]])
def test_few_tokens_of_wide_rows_are_requested_ahead_of_the_normalisation(record, dtype, T, d, E, norm, ahead):
    (rc, found), = record(route_call(T, d, E, 2, dtype, norm))
    assert rc == 0 and found[0].kernel.startswith("route_small_tokens") and found[0].kernel.endswith(f", {ahead}>")


@pytest.mark.parametrize("dtype,T,d,E,waves", [
    (B.BTX_BF16, 4097, 4096, 16, 8), (B.BTX_BF16, 4097, 4096, 17, 4), (B.BTX_BF16, 4097, 4104, 17, 8), (B.BTX_BF16, 8176, 10240, 32, 8),
    (B.BTX_BF16, 8176, 10248, 17, 4), (B.BTX_BF16, 8176, 16384, 16, 8), (B.BTX_BF16, 8177, 16384, 16, 4), (B.BTX_BF16, 4097, 8192, 33, 4),
    (B.BTX_F32, 4097, 4104, 16, 8), (B.BTX_F32, 4097, 4104, 17, 4)])
def test_wide_rows_share_their_tokens_between_8_wavefronts(record, dtype, T, d, E, waves):
    (rc, found), = record(route_call(T, d, E, 2, dtype))
    tokens, = [launch for launch in found if launch.kernel.startswith("route_tokens")]
    assert rc == 0 and tokens.block[0] == 64 * waves


@pytest.mark.parametrize("dtype", [B.BTX_F32, B.BTX_BF16])
@pytest.mark.parametrize("E", [1, 2, 3, 4, 5, 8, 9, 12, 16, 17, 64])
def test_routing_takes_the_same_way_with_and_without_the_normalisation(record, E, dtype):
    """btx_moe_norm_route routes exactly as btx_moe_route does from the rows it wrote: few tokens go to the same kernels in both, as
    the kernels for few and for many tokens add up a logit in different orders."""
    shapes = [(T, d) for T in (1, 500, 512, 513, 600, 640, 641, 750, 1000, 1024, 1025) for d in (64, 256, 512, 1024, 1040, 2048, 2936, 4096, 8192)]
    found = record(*(route_call(T, d, E, min(E, 2), dtype, norm) for T, d in shapes for norm in (False, True)))
    for shape, (rc, plain), (norm_rc, norm) in zip(shapes, found[::2], found[1::2]):
        assert rc == norm_rc == 0
        assert ("route_small" in plain[0].kernel) == ("route_small" in norm[0].kernel), shape


@pytest.mark.parametrize("case,taken", ROUTE_MANY)
def test_shapes_of_many_tokens_routing_take_that_path(record, case, taken):
    T, d, E, k, dtype, norm = case
    (rc, found), = record(route_call(*case))
    tokens, = [launch.kernel for launch in found if launch.kernel.startswith("route_tokens")]
    experts, with_norm, waves = re.search(r", (\d+), (true|false), (\d+), ", tokens).groups()
    assert rc == 0 and (int(experts), int(waves)) == taken and with_norm == str(norm).lower()


@pytest.mark.parametrize("T,d,E,k,launches", [
    (512, 4096, 5, 2, 2), (512, 8192, 8, 2, 2), (512, 8200, 8, 2, 4),
    # above 512 tokens: whole vector loads of W_router
    (1024, 1024, 4, 2, 2), (732, 4096, 4, 2, 2), (733, 4096, 4, 2, 4), (1025, 64, 4, 2, 4), (640, 64, 4, 4, 2), (641, 64, 4, 4, 4), (640, 2336, 8, 2, 2),
    (640, 2352, 8, 2, 4), (641, 64, 8, 2, 4), (640, 1024, 16, 4, 2), (520, 1032, 16, 4, 4), (640, 1816, 9, 2, 2), (640, 1832, 9, 2, 4),
    # columns of W_router that are loaded one by one
    (1024, 4096, 1, 1, 4), (1024, 480, 1, 1, 2), (1024, 512, 2, 2, 4), (1024, 384, 2, 2, 2), (1024, 1024, 3, 2, 4), (600, 256, 3, 2, 2), (520, 4096, 5, 2, 4),
    (640, 2048, 5, 2, 4), (640, 400, 5, 2, 2), (640, 416, 5, 2, 4), (640, 176, 7, 2, 2), (640, 448, 7, 2, 4), (640, 1536, 12, 4, 4), (640, 256, 15, 4, 2), (640, 1024, 14, 4, 4), (513, 64, 17, 2, 4)])
@pytest.mark.parametrize("norm", [False, True])
def test_routing_launches(record, T, d, E, k, launches, norm):
    (rc, found), = record(route_call(T, d, E, k, B.BTX_BF16, norm))
    assert rc == 0 and len(found) == launches


@pytest.mark.parametrize("dtype,T,d,f,E,k,sliced", [
    (B.BTX_BF16, 16, 4096, 11008, 4, 2, True), (B.BTX_BF16, 40, 512, 5504, 8, 4, True), (B.BTX_BF16, 100, 512, 1376, 16, 8, True),
    (B.BTX_F32, 64, 512, 1376, 8, 8, True), (B.BTX_F32, 10, 128, 1024, 16, 8, True),
    # too many slices of too many slots; slots that are looked up as they come; products that are not cut
    (B.BTX_BF16, 40, 512, 5504, 8, 5, False), (B.BTX_BF16, 40, 512, 5504, 8, 8, False), (B.BTX_BF16, 7, 256, 4096, 12, 12, False),
    (B.BTX_F32, 10, 128, 1024, 16, 12, False), (B.BTX_BF16, 301, 4096, 11008, 4, 2, False), (B.BTX_F32, 2003, 512, 1376, 8, 2, False)])
def test_slices_of_the_down_projection_are_added_once(record, dtype, T, d, f, E, k, sliced):
    """By the combine, or by a finishing kernel of the product."""
    (rc, found), = record(forward_call(T, d, f, E, k, dtype))
    names = [launch.kernel for launch in found]
    assert rc == 0 and names[-1].startswith("combine_kernel") and names[-1].endswith("true>") == sliced
    if sliced:
        assert "finish" not in names[-2]
    elif T < 100:
        assert "slices_finish" in names[-2]


@pytest.mark.parametrize("T,d,f,E,kw,streamed", [
    # rows per expert: what a tile of 64, 128 (96), 192 and 256 (236) rows has room for
    (4 * 48, 4096, 11008, 4, {}, "UP DOWN"), (4 * 96, 4096, 11008, 4, {}, "UP DOWN"), (4 * 97, 4096, 11008, 4, {}, ""), (4 * 111, 4096, 11008, 4, {}, "UP DOWN"),
    (4 * 168, 4096, 11008, 4, {}, "UP DOWN"), (4 * 236, 4096, 11008, 4, {}, "UP DOWN"), (4 * 237, 4096, 11008, 4, {}, ""),
    # 300 million bytes of weights
    (16, 3072, 5504, 3, {}, "UP DOWN"), (16, 2560, 6528, 3, {}, "UP DOWN"), (16, 2560, 6464, 3, {}, ""), (16, 2048, 5504, 4, {}, ""),
    # rows of whole lines, from the first expert's to the last one's
    (16, 4096, 11008, 4, dict(p=P + 64), ""), (16, 4096, 11008, 4, dict(stride=4096 * 11008 + 32), ""), (16, 4096, 11008, 4, dict(stride=4096 * 11008 + 64), "UP DOWN"),
    # K of whole k tiles, rows of whole lines: W2 has K = f rows of d columns
    (16, 4096, 11040, 4, {}, ""), (16, 4096, 688, 64, {}, ""), (16, 4128, 11008, 4, {}, ""), (64, 1024, 2752, 32, {}, "UP DOWN")])
def test_weights_are_streamed_where_they_are_read_once(record, T, d, f, E, kw, streamed):
    (rc, found), = record(forward_call(T, d, f, E, 1, B.BTX_BF16, **kw))
    assert rc == 0
    for launch in found:
        if launch.kernel.startswith("mfma_small"):
            *numbers, stream = launch.kernel[:-1].split(", ")
            product = int(numbers[5])
        elif launch.kernel.startswith("mfma_gemm"):
            *numbers, stream, _ = launch.kernel[:-1].split(", ")
            product = int(numbers[7])
        else:
            continue
        assert (stream == "true") == ({UP: "UP", DOWN: "DOWN"}[product] in streamed.split()), launch.kernel


@pytest.mark.parametrize("T,d,f,E,product,tile", [
    # one round of 256- or 192-row tiles where smaller ones would need a second round (us there: 256 / 128 rows)
    (400, 4096, 11008, 2, UP, 256), (480, 4096, 11008, 1, UP, 256), (6000, 4096, 688, 4, UP, 256), (320, 4096, 11008, 2, UP, 192),
    (2300, 4096, 11008, 1, DOWN, 256), (600, 2048, 5504, 1, BWD_DX, 256), (4600, 2048, 5504, 2, BWD_DX, 256), (2300, 8192, 4096, 1, BWD_ACT, 256),
    # compute units that large tiles would leave idle
    (1200, 4096, 1376, 4, BWD_DX, 128), (1200, 4096, 1376, 4, DOWN, 128), (1200, 4096, 1376, 4, BWD_ACT, 64), (600, 512, 1376, 4, UP, 64),
    # enough large tiles
    (16384, 4096, 11008, 4, DOWN, 256), (4001 * 2, 2048, 5504, 8, BWD_DX, 256)])
def test_row_tiles_of_products_with_few_tiles(record, T, d, f, E, product, tile):
    assert bf16_products(record, T, d, f, E, 1)[product][0] == tile
