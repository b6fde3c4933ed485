"""GPU parity tests: the HIP library, called through its C ABI, against the CPU
oracle on the same seeded inputs, element by element."""
import numpy as np
import pytest
import torch

from oracle import btx_oracle as O
from paper_2403_07816_amd import binding as B
from paper_2403_07816_amd import synth

from conftest import assert_close
from helpers import TOL, as_passed, run_block_and_check, run_layer_and_check, to_dev, to_np, experts_np, check_route
from path_cases import (DY_ROWS, DY_TRANSPOSED, F32_LAST_ROUND, FEW_K_TILES, JOINT_FORWARD, LAST_ROUND_CUT, ROUTE_AHEAD, ROUTE_MANY, ROW_PITCH, TILED_FORWARD,
                        TRANSPOSED_ROWS, WHOLE_TILE_CASES, whole_tile_case)

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16


# ------------------------------------------------------------------ fp32 path
def test_config0_tiny_fp32_forward():
    """T=512, d=64, f=176, E=4, top-2, fp32, forward only."""
    run_layer_and_check(512, 64, 176, 4, 2, F32, backward=False)


def test_config0_shape_fp32_forward_backward():
    run_layer_and_check(512, 64, 176, 4, 2, F32)


@pytest.mark.parametrize("T,d,f,E,k", [(301, 72, 88, 5, 3), (1, 64, 64, 4, 2), (67, 136, 200, 7, 7), (130, 64, 40, 32, 8),
                                       (1000, 128, 64, 64, 4), (17, 8, 8, 1, 1),
                                       # expert counts that leave the last register chunk of the router kernels
                                       # partly empty (8 per pass forward, 16 in the backward)
                                       (45, 64, 64, 33, 5), (300, 128, 96, 17, 3), (257, 72, 40, 9, 9),
                                       # more than 8 experts: router logits from the matrix cores, 16 experts per
                                       # set (3 sets here), rows that end inside a 32-column piece
                                       (2000, 200, 64, 48, 6)])
def test_ragged_shapes_fp32(T, d, f, E, k):
    run_layer_and_check(T, d, f, E, k, F32)


@pytest.mark.parametrize("T,d,f,E,k,kw", [(4000, 1032, 1160, 8, 2, {}), (4000, 1160, 1032, 8, 2, dict(cf=0.8, poison=True)),
                                          (129, 8, 136, 2, 1, {}), (130, 136, 8, 3, 2, dict(poison=True)),
                                          (257, 72, 184, 4, 3, {})])
def test_fp32_tiles(T, d, f, E, k, kw):
    """The fp32 products: many and few tiles, ragged rows, columns and contractions, token rows read through perm."""
    run_layer_and_check(T, d, f, E, k, F32, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", [(64, 512, 1376, 8, 2, {}), (40, 72, 1032, 4, 2, {}), (1, 64, 2056, 3, 2, {}),
                                          (130, 136, 776, 4, 2, dict(cf=0.8, poison=True)), (300, 264, 1384, 2, 1, {})])
def test_fp32_products_cut_along_k(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, F32, **kw)


@pytest.mark.parametrize("T,d,f,E,k", [(1, 680, 8192, 2, 2), (12, 5528, 216, 16, 2), (100, 4104, 344, 8, 1), (37, 3984, 216, 16, 2), (65, 2800, 4096, 1, 1)])
def test_fp32_up_projection_with_three_stages(T, d, f, E, k):
    """Last k tiles of 8, 16, 24 and 32, 22 to 173 of them, one and two row tiles to an expert."""
    run_layer_and_check(T, d, f, E, k, F32, unit_rms=True, backward=False, poison=True)


@pytest.mark.parametrize("T,d,f,E,k,kw", JOINT_FORWARD)
def test_fp32_small_layers_forward_in_one_launch(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, F32, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", [case for case, _ in TILED_FORWARD])
def test_fp32_forward_of_narrow_rows_in_two_launches(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, F32, backward=False, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", F32_LAST_ROUND)
def test_fp32_last_round_of_the_down_projection_cut_along_k(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, F32, backward=False, poison=True, **kw)


def test_fp32_token_rows_past_4_gib():
    """Token rows whose byte offsets need more than 32 bits: as the same rows give in batches that stay below.  Without a
    load-balancing loss the tokens do not see each other; the weight gradients add up."""
    T, d, f, E = (1 << 17) + 104, 1 << 13, 16, 2
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dY = (torch.randn((T, d), generator=g, device="cuda") for _ in range(2))
    W1, W3 = (torch.randn((E, d, f), generator=g, device="cuda") / d ** 0.5 for _ in range(2))
    W2, Wr = torch.randn((E, f, d), generator=g, device="cuda") / f ** 0.5, torch.randn((d, E), generator=g, device="cuda") * 0.02

    def step(x, dY):
        r = B.btx_moe_route(x, Wr, None, None, 1, B.BTX_ROUTE_SWITCH_TOP1)
        out, h1, h3 = B.btx_moe_ff_forward(x, W1, W3, W2, r)
        b = B.btx_moe_ff_backward(dY, x, Wr, W1, W3, W2, r, h1, h3, B.BTX_ROUTE_SWITCH_TOP1)
        return out, b.dX, [t.double() for t in (b.dW1, b.dW3, b.dW2, b.dW_router)]

    out, dX, sums = step(x, dY)
    parts = [0.0] * len(sums)
    for at in range(0, T, T // 4):
        rows = slice(at, at + T // 4)
        part_out, part_dX, dW = step(x[rows], dY[rows])
        # fp32 sums of at most 8192 terms, each in the order of the whole batch; the routing's of any order
        for got, want in ((out[rows], part_out), (dX[rows], part_dX)):
            assert float((got - want).norm() / want.norm()) < 1e-6
        parts = [a + b for a, b in zip(parts, dW)]
    for got, want in zip(sums, parts):          # 65 thousand terms of random signs, in two orders
        assert float((got - want).norm() / want.norm()) < TOL[F32] / 4


@pytest.mark.parametrize("T,d,f,pieces", [(257, 264, 8421504, 16), (66, 136, 34087048, 56)])
def test_bf16_experts_whose_rows_need_64_bit_offsets(T, d, f, pieces):
    """256 rows of f elements, or 64 of them, span 4 GiB: the down-projection and the input gradient (and the up-projection with 64 rows of
    its weights) find them with 64-bit offsets.  One expert, whose gate is 1; against fp32 products, a piece of the columns at a time."""
    g = torch.Generator(device="cuda").manual_seed(6)
    def draw(*shape, scale=1.0):
        return torch.randn(shape, generator=g, device="cuda", dtype=BF16).mul_(scale)
    x, dY, W1, W3, W2 = draw(T, d), draw(T, d), draw(1, d, f, scale=d ** -0.5), draw(1, d, f, scale=d ** -0.5), draw(1, f, d, scale=f ** -0.5)
    Wr = torch.zeros((d, 1), device="cuda")
    r = B.btx_moe_route(x, Wr, None, None, 1, B.BTX_ROUTE_SWITCH_TOP1)
    out, h1, h3 = B.btx_moe_ff_forward(x, W1, W3, W2, r)
    b = B.btx_moe_ff_backward(dY, x, Wr, W1, W3, W2, r, h1, h3, B.BTX_ROUTE_SWITCH_TOP1)

    def check(got, want, what):
        err = float((got.float() - want).norm() / want.norm())
        assert err < TOL[BF16], f"{what}: {err:.2e}"
    rows = torch.argsort(r.inv_pos.flatten().long())                # grouped row -> token
    xf, dYf = x.float()[rows], dY.float()[rows]
    want_out, want_dX = torch.zeros((T, d), device="cuda", dtype=torch.float64), torch.zeros((T, d), device="cuda", dtype=torch.float64)
    for p in range(pieces):
        c = slice(p * f // pieces, (p + 1) * f // pieces)
        w1, w3, w2 = W1[0, :, c].float(), W3[0, :, c].float(), W2[0, c].float()
        u1, u3 = xf @ w1, xf @ w3
        check(h1[:, c], u1, f"h1, piece {p}")
        check(h3[:, c], u3, f"h3, piece {p}")
        want_out += ((torch.nn.functional.silu(u1) * u3).to(BF16).float() @ w2).double()
        u1, u3 = h1[:, c].float(), h3[:, c].float()
        s = torch.sigmoid(u1)
        da = dYf @ w2.t().contiguous()
        dh1, dh3, ga = ((v.to(BF16).float()) for v in (da * u3 * s * (1 + u1 * (1 - s)), da * u1 * s, u1 * s * u3))
        want_dX += (dh1 @ w1.t().contiguous()).double() + (dh3 @ w3.t().contiguous()).double()
        check(b.dW1[0, :, c], xf.t().contiguous() @ dh1, f"dW1, piece {p}")
        check(b.dW3[0, :, c], xf.t().contiguous() @ dh3, f"dW3, piece {p}")
        check(b.dW2[0, c], ga.t().contiguous() @ dYf, f"dW2, piece {p}")
    check(out[rows], want_out, "out")
    check(b.dX[rows], want_dX, "dX")
    del out, h1, h3, b, W1, W3, W2
    torch.cuda.empty_cache()


def test_bf16_token_rows_that_need_64_bit_offsets():
    """255 token rows of d elements would span 4 GiB: the up-projection and the activation's gradient run with 64-bit offsets.  Otherwise as above."""
    T, d, f, pieces = 70, 8421504, 72, 16
    g = torch.Generator(device="cuda").manual_seed(7)
    def draw(*shape, scale=1.0):
        return torch.randn(shape, generator=g, device="cuda", dtype=BF16).mul_(scale)
    x, dY, W1, W3, W2 = draw(T, d), draw(T, d), draw(1, d, f, scale=d ** -0.5), draw(1, d, f, scale=d ** -0.5), draw(1, f, d, scale=f ** -0.5)
    r = B.btx_moe_route(x, torch.zeros((d, 1), device="cuda"), None, None, 1, B.BTX_ROUTE_SWITCH_TOP1)
    out, h1, h3 = B.btx_moe_ff_forward(x, W1, W3, W2, r)
    b = B.btx_moe_ff_backward(dY, x, torch.zeros((d, 1), device="cuda"), W1, W3, W2, r, h1, h3, B.BTX_ROUTE_SWITCH_TOP1)

    def check(got, want, what):
        err = float((got.float() - want).norm() / want.norm())
        assert err < TOL[BF16], f"{what}: {err:.2e}"
    rows = torch.argsort(r.inv_pos.flatten().long())                # grouped row -> token
    columns = [slice(p * d // pieces, (p + 1) * d // pieces) for p in range(pieces)]
    want1, want3, da = (torch.zeros((T, f), device="cuda", dtype=torch.float64) for _ in range(3))
    for c in columns:
        xf, dYf = x[:, c].float()[rows], dY[:, c].float()[rows]
        want1 += (xf @ W1[0, c].float()).double()
        want3 += (xf @ W3[0, c].float()).double()
        da += (dYf @ W2[0, :, c].float().t().contiguous()).double()
    check(h1, want1, "h1")
    check(h3, want3, "h3")
    u1, u3 = h1.float(), h3.float()
    s = torch.sigmoid(u1)
    act, dh1, dh3 = (v.to(BF16).float() for v in (u1 * s * u3, da.float() * u3 * s * (1 + u1 * (1 - s)), da.float() * u1 * s))
    for p, c in enumerate(columns):
        w1, w3, xf, dYf = W1[0, c].float(), W3[0, c].float(), x[:, c].float()[rows], dY[:, c].float()[rows]
        check(out[:, c][rows], act @ W2[0, :, c].float(), f"out, piece {p}")
        check(b.dX[:, c][rows], dh1 @ w1.t().contiguous() + dh3 @ w3.t().contiguous(), f"dX, piece {p}")
        check(b.dW1[0, c], xf.t().contiguous() @ dh1, f"dW1, piece {p}")
        check(b.dW3[0, c], xf.t().contiguous() @ dh3, f"dW3, piece {p}")
        check(b.dW2[0, :, c], act.t().contiguous() @ dYf, f"dW2, piece {p}")


@pytest.mark.parametrize("mode", [B.BTX_ROUTE_SWITCH_TOP1, B.BTX_ROUTE_SAMPLE_TOP1])
@pytest.mark.parametrize("lb_mode,flags", [(B.BTX_LB_TOKEN_FRAC, 0), (B.BTX_LB_GATE_MEAN, 0),
                                           (B.BTX_LB_GATE_MEAN, B.BTX_FLAG_LB_GRAD_THROUGH_U)])
def test_top1_variants_with_biased_router_fp32(mode, lb_mode, flags):
    run_layer_and_check(700, 64, 96, 4, 1, F32, mode=mode, lb_mode=lb_mode, flags=flags, bias=[2.0, 0, 0, 0],
                        alpha=0.5)


@pytest.mark.parametrize("mode", [B.BTX_ROUTE_SWITCH_TOP1, B.BTX_ROUTE_SAMPLE_TOP1, B.BTX_ROUTE_GUMBEL_TOP1])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_top1_variants_with_many_experts(mode, dtype):
    """The top-1 selections on logits that come from the matrix cores (more than 8 experts)."""
    bias = [1.5, 0, 0, -0.5, 0, 0, 0.5, 0, 0, 0, 0, 0]
    run_layer_and_check(500, 160, 96, 12, 1, dtype, mode=mode, bias=bias, unit_rms=(dtype == BF16), tau=0.7)


@pytest.mark.parametrize("lb_mode,flags,lam", [(B.BTX_LB_TOKEN_FRAC, 0, 1.0), (B.BTX_LB_GATE_MEAN, 0, 1.0),
                                               (B.BTX_LB_GATE_MEAN, B.BTX_FLAG_LB_GRAD_THROUGH_U, 2.0),
                                               (B.BTX_LB_TOKEN_FRAC, 0, 0.0)])
def test_topk_load_balancing_variants_fp32(lb_mode, flags, lam):
    # alpha is large so that the load-balancing gradient is visible next to the main one
    run_layer_and_check(600, 64, 96, 6, 2, F32, lb_mode=lb_mode, flags=flags, lam=lam, alpha=5.0)


@pytest.mark.parametrize("tau", [1.0, 0.5, 3.0])
@pytest.mark.parametrize("lb_mode,flags", [(B.BTX_LB_TOKEN_FRAC, 0), (B.BTX_LB_GATE_MEAN, B.BTX_FLAG_LB_GRAD_THROUGH_U)])
def test_gumbel_sample_top1_fp32(tau, lb_mode, flags):
    run_layer_and_check(301, 72, 88, 5, 1, F32, mode=B.BTX_ROUTE_GUMBEL_TOP1, lb_mode=lb_mode, flags=flags,
                        bias=[0.5, 0, -0.5, 0, 0.2], tau=tau)


def test_gumbel_at_vanishing_temperature_is_the_hard_sample():
    """tau -> 0+: the soft sample becomes one-hot, i.e. the inference-time hard sampling (gate 1)."""
    L = synth.make_layer(300, 64, 64, 4, dtype=F32, with_gumbel=True)
    G = to_dev(L)
    r = B.btx_moe_route(G["x"], G["W_router"], None, G["U"], 1, B.BTX_ROUTE_GUMBEL_TOP1, tau=1e-4)
    noisy = O.router_logits(to_np(L["x"]), to_np(L["W_router"])) + to_np(L["U"])
    gap = np.sort(noisy, axis=1)
    clear = (gap[:, -1] - gap[:, -2]) > 1e-2
    assert clear.sum() > 250
    assert np.array_equal(r.topk_idx.cpu().numpy()[clear, 0], np.argmax(noisy, axis=1)[clear])
    assert np.all(r.gates.cpu().numpy()[clear, 0] == 1.0)


def test_gumbel_without_noise_at_unit_temperature_is_switch_routing():
    L = synth.make_layer(257, 64, 64, 4, dtype=F32, with_dY=True)
    G = to_dev(L)
    zero = torch.zeros((257, 4), device="cuda")
    a = B.btx_moe_route(G["x"], G["W_router"], None, zero, 1, B.BTX_ROUTE_GUMBEL_TOP1, tau=1.0)
    b = B.btx_moe_route(G["x"], G["W_router"], None, None, 1, B.BTX_ROUTE_SWITCH_TOP1)
    assert torch.equal(a.topk_idx, b.topk_idx) and torch.equal(a.perm, b.perm)
    assert_close(a.gates.cpu().numpy(), b.gates.cpu().numpy().astype(np.float64), 1e-6, "gates")


@pytest.mark.parametrize("mode,k,cf,bias", [(B.BTX_ROUTE_SWITCH_TOP1, 1, 1.5, [2.0, 0, 0, 0]),
                                            (B.BTX_ROUTE_SWITCH_TOP1, 1, 0.5, None),
                                            (B.BTX_ROUTE_TOPK_RENORM, 2, 0.75, [1.0, 0, 0, -1.0]),
                                            (B.BTX_ROUTE_TOPK_RENORM, 2, 4.0, None)])
def test_capacity_factor_drops_pairs_in_token_order_fp32(mode, k, cf, bias):
    G, r, out, g = run_layer_and_check(301, 72, 88, 4, k, F32, mode=mode, bias=bias, cf=cf)
    dropped = int((r.inv_pos < 0).sum())
    assert (dropped > 0) == (cf < 4.0)
    assert int(r.offsets[-1]) == 301 * k - dropped


def test_capacity_factor_with_many_experts_fp32():
    """Dropped pairs where the router backward reloads its W_router slice in chunks (E > 16)."""
    G, r, out, g = run_layer_and_check(400, 64, 64, 24, 4, F32, cf=0.5, bias=[1.0] * 4 + [0.0] * 20)
    assert int((r.inv_pos < 0).sum()) > 0


def test_capacity_factor_gate_mean_statistics_fp32():
    # (capacity factors in these tests are exact in binary: the C ABI takes a float)
    run_layer_and_check(257, 64, 64, 4, 2, F32, lb_mode=B.BTX_LB_GATE_MEAN, flags=B.BTX_FLAG_LB_GRAD_THROUGH_U,
                        bias=[1.5, 0, 0, 0], cf=0.625)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_residual_is_added_in_the_combine(dtype):
    """out = residual + FF_MoE(x) in one pass, one rounding; with a capacity limit the tokens that lost
    all their pairs come out as the residual alone."""
    T, d, f, E = 333, 128, 192, 4
    L = synth.make_layer(T, d, f, E, dtype=dtype, unit_rms=True, router_bias=[2.0, 0, 0, 0])
    G = to_dev(L)
    res = (torch.randn(T, d, generator=torch.Generator().manual_seed(5)) * 2).to(dtype)
    r = B.btx_moe_route(G["x"], G["W_router"], G["b_router"], None, 1, B.BTX_ROUTE_SWITCH_TOP1, capacity_factor=1.0)
    fwd = check_route(r, L, 1, B.BTX_ROUTE_SWITCH_TOP1, 0.0, B.BTX_LB_TOKEN_FRAC, cf=1.0)
    out, _, _ = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r, save=False, residual=res.cuda())
    assert_close(to_np(out), fwd["out"] + to_np(res), TOL[dtype], "residual + out")
    lost = fwd["dropped"][:, 0]
    assert lost.any() and torch.equal(out.cpu()[torch.from_numpy(lost)], res[torch.from_numpy(lost)])


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_residual_may_be_x_or_the_output_buffer_and_db_router_may_be_left_out(dtype):
    """The aliasing the header allows: residual = x (h + FF(h) with h both routed and added) and
    residual = out (the sum lands on top of the residual), each bit for bit what separate buffers give;
    db_router = NULL leaves every other gradient as it is."""
    T, d, f, E, k = 257, 128, 192, 4, 2
    L = synth.make_layer(T, d, f, E, dtype=dtype, unit_rms=True, with_dY=True)
    G = to_dev(L)
    r = B.btx_moe_route(G["x"], G["W_router"], None, None, k)
    want, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r, residual=G["x"].clone())
    same_x, _, _ = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r, residual=G["x"])
    assert torch.equal(same_x, want)
    buf = G["x"].clone()
    B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r, out=buf, residual=buf)
    assert torch.equal(buf, want)
    full = B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3)
    part = B.Grads(torch.empty_like(full.dX), torch.empty_like(full.dW_router), None, torch.empty_like(full.dW1),
                   torch.empty_like(full.dW3), torch.empty_like(full.dW2))
    B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3, out=part)
    for a, b in ((part.dX, full.dX), (part.dW_router, full.dW_router), (part.dW1, full.dW1), (part.dW2, full.dW2)):
        assert torch.equal(a, b)


def test_expert_without_tokens_fp32():
    """A strongly negative bias starves expert 2: empty group, zero weight gradients."""
    G, r, out, g = run_layer_and_check(300, 64, 80, 4, 2, F32, bias=[0, 0, -60.0, 0])
    assert r.counts.cpu().numpy()[2] == 0


def test_soft_routing_all_experts_active_fp32():
    run_layer_and_check(200, 64, 48, 4, 4, F32)


def test_split_experts_fp32():
    """Each of 2 FFNs cut into 4 chunks: 8 experts of a quarter width, top-4."""
    run_layer_and_check(256, 64, 32, 8, 4, F32, split=4)


def test_identical_experts_equal_dense_ff_on_gpu():
    """Sparse-upcycling special case: the MoE output equals the dense seed FF and
    dW_router vanishes when load balancing is off."""
    G, r, out, g = run_layer_and_check(400, 64, 96, 4, 2, F32, identical=True, lam=0.0, check_router_grads=False)
    x = to_np(G["x"])
    W1, W3, W2 = (to_np(G[n][0]) for n in ("W1", "W3", "W2"))
    h1 = x @ W1
    dense = (h1 / (1 + np.exp(-h1)) * (x @ W3)) @ W2
    assert_close(to_np(out), dense, 1e-4, "dense FF")
    assert np.abs(to_np(g.dW_router)).max() < 1e-4 * np.abs(to_np(g.dX)).max() * 400


def test_results_are_bit_identical_run_to_run():
    L = to_dev(synth.make_layer(777, 128, 192, 8, dtype=F32, with_dY=True))
    outs = []
    for _ in range(2):
        r = B.btx_moe_route(L["x"], L["W_router"], None, None, 2, lb_alpha=0.01)
        out, h1, h3 = B.btx_moe_ff_forward(L["x"], L["W1"], L["W3"], L["W2"], r)
        g = B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3, lb_alpha=0.01,
                                  lb_grad_scale=1.0)
        outs.append([t.clone() for t in (r.perm, r.gates, r.lb_loss, out, g.dX, g.dW_router, g.dW1, g.dW2, g.dW3)])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,d,f", [(BF16, 128, 160), (BF16, 72, 264), (F32, 64, 176)])
def test_expert_matrices_with_padding_between_them(dtype, d, f):
    """Stacked expert weights whose experts lie further apart than d*f elements (the strides are arguments of
    the C ABI), gradients returned with the same strides: bit for bit what the packed tensors give, and the
    padding is left alone."""
    T, E, k, pad = 300, 3, 2, 24
    L = synth.make_layer(T, d, f, E, dtype=dtype, unit_rms=(dtype == BF16), with_dY=True)
    G = to_dev(L)

    def padded(W, fill):
        base = torch.full((E, W.shape[1] * W.shape[2] + pad), fill, dtype=W.dtype, device="cuda")
        view = base[:, :W.shape[1] * W.shape[2]].view(E, W.shape[1], W.shape[2])
        return base, view
    P = {}
    for n in ("W1", "W3", "W2"):
        base, view = padded(G[n], float("nan"))
        view.copy_(G[n])
        P[n] = view
    r = B.btx_moe_route(G["x"], G["W_router"], None, None, k, lb_alpha=0.01)
    out0, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r)
    out1, g1, g3 = B.btx_moe_ff_forward(G["x"], P["W1"], P["W3"], P["W2"], r)
    assert torch.equal(out0, out1) and torch.equal(h1, g1) and torch.equal(h3, g3)
    want = B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3, lb_alpha=0.01,
                                 lb_grad_scale=1.0)
    bases, views = zip(*(padded(G[n], 7.0) for n in ("W1", "W3", "W2")))
    got = B.Grads(torch.empty_like(G["x"]), torch.empty_like(want.dW_router), torch.empty_like(want.db_router), *views)
    B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], P["W1"], P["W3"], P["W2"], r, h1, h3, lb_alpha=0.01,
                          lb_grad_scale=1.0, out=got)
    assert torch.equal(got.dX, want.dX) and torch.equal(got.dW_router, want.dW_router)
    for a, b in ((got.dW1, want.dW1), (got.dW3, want.dW3), (got.dW2, want.dW2)):
        assert torch.equal(a, b)
    for base, W in zip(bases, (G["W1"], G["W3"], G["W2"])):
        assert bool((base[:, W.shape[1] * W.shape[2]:] == 7.0).all())


def test_frozen_experts_skip_weight_gradients():
    L = to_dev(synth.make_layer(200, 64, 96, 4, dtype=F32, with_dY=True))
    r = B.btx_moe_route(L["x"], L["W_router"], None, None, 2)
    out, h1, h3 = B.btx_moe_ff_forward(L["x"], L["W1"], L["W3"], L["W2"], r)
    full = B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3)
    frozen = B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3,
                                   frozen_experts=True)
    assert frozen.dW1 is None
    assert torch.equal(full.dX, frozen.dX) and torch.equal(full.dW_router, frozen.dW_router)


@pytest.mark.parametrize("T,d,f,E,k", [(1, 8, 8, 4, 1), (65, 72, 136, 3, 2), (64, 512, 1376, 8, 2), (1501, 136, 1032, 5, 2)])
def test_fp32_gradients_of_frozen_and_trained_experts(T, d, f, E, k):
    """The products of the backward pass in one launch: few and many tiles of each, cut along K and not; the input's gradients are
    those of the product alone, the weights' those of the oracle."""
    run_layer_and_check(T, d, f, E, k, F32, poison=True)
    L = to_dev(synth.make_layer(T, d, f, E, dtype=F32, with_dY=True))
    r = B.btx_moe_route(L["x"], L["W_router"], None, None, k)
    _, h1, h3 = B.btx_moe_ff_forward(L["x"], L["W1"], L["W3"], L["W2"], r)
    full, frozen = (B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3, frozen_experts=z)
                    for z in (False, True))
    assert torch.equal(full.dX, frozen.dX) and torch.equal(full.dW_router, frozen.dW_router)


def test_empty_batch_is_a_noop():
    x = torch.empty((0, 64), device="cuda")
    Wr = torch.zeros((64, 4), device="cuda")
    r = B.btx_moe_route(x, Wr, None, None, 2)
    assert r.topk_idx.shape == (0, 2)


# ------------------------------------------------------------------ bf16 path
@pytest.mark.parametrize("T,d,f,E,k", [(512, 256, 384, 4, 2), (333, 264, 200, 4, 2), (1500, 512, 1376, 8, 4),
                                       (40, 64, 72, 4, 1),
                                       # the products at their edges: fewer rows than one k tile, many (mostly tiny or
                                       # empty) experts, d and f that are multiples of 32 but not of 64
                                       (5, 64, 64, 4, 2), (700, 96, 160, 64, 8), (257, 320, 96, 3, 3),
                                       (300, 128, 96, 17, 3)])
def test_bf16_forward_backward(T, d, f, E, k):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True)


@pytest.mark.parametrize("T,d,f,E,k", [(313, 120, 264, 4, 2), (200, 264, 520, 3, 1), (150, 72, 776, 5, 3)])
def test_bf16_widths_off_the_32_grid_with_wide_experts(T, d, f, E, k):
    """d or f not a multiple of 32, and f > 256: several column tiles, the last one partial, each with its own sum of D * act."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True)


@pytest.mark.parametrize("T,d,f,E,k", [(70, 8, 8, 2, 1), (300, 56, 40, 3, 2), (261, 72, 88, 4, 2), (190, 104, 120, 5, 3),
                                       # K slices of small tiles that end in a partial k tile (f, d = 40, 8 mod 64)
                                       (700, 328, 2088, 3, 2), (300, 1096, 312, 2, 1)])
def test_bf16_contractions_that_end_inside_a_k_tile(T, d, f, E, k):
    """d and f that are multiples of 8 only: the last k tile holds 1 to 7 chunks of 8, in both operand layouts."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True)


def _random_small_tile_case(i):
    rng = np.random.default_rng(1000 + i)
    E = int(rng.choice([1, 2, 3, 4, 6, 8, 16]))
    k = int(rng.integers(1, min(E, 4) + 1))
    d = 32 * int(rng.integers(2, 13))
    f = 32 * int(rng.integers(2, 20))
    T = int(rng.integers(1, 1200))
    return T, d, f, E, k


@pytest.mark.parametrize("case", range(12))
def test_bf16_random_shapes_of_small_tiles(case):
    """Seeded random shapes (d, f multiples of 32; 1-16 experts; ragged groups of every size): 64- and 128-row tiles,
    tile edges, padded groups, last k tiles that are half full."""
    T, d, f, E, k = _random_small_tile_case(case)
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, seed=synth.BASE_SEED + case,
                        dW_dtype=F32 if case % 3 == 0 else None)


@pytest.mark.parametrize("case", range(WHOLE_TILE_CASES))
def test_bf16_random_shapes_of_whole_tiles(case):
    """Seeded random shapes large enough for 256-row tiles in all four row-grouped products: partial row and column tiles,
    ragged strips of the tile order, every form of the last k tile."""
    T, d, f, E, k = whole_tile_case(case)
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, seed=synth.BASE_SEED + case)


@pytest.mark.parametrize("case,products", FEW_K_TILES)
def test_bf16_few_k_tiles_of_large_row_tiles(case, products):
    T, d, f, E, k, options = case
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True, **options)


@pytest.mark.parametrize("case,paths", LAST_ROUND_CUT)
def test_bf16_last_round_cut_along_k(case, paths):
    """256- and 192-row tiles of a partly filled last round in K ranges of their own, whose sums a second kernel adds: every product
    that is cut, every form of the last k tile, dropped pairs.  That the shapes take these paths is checked on the CPU."""
    T, d, f, E, k, options = case
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True, **options)


@pytest.mark.parametrize("T,d,f,E,k,kw", [
    (700, 320, 2080, 3, 2, {}),
    # top-1 with dropped pairs: rows of the output nothing writes, tiles of unequal height
    (900, 256, 2048, 4, 1, dict(mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[2.0, 0, 0, 0], cf=1.5)),
    (600, 4096, 1024, 3, 2, {}),
    (1100, 4096, 1024, 4, 2, {}),
])
def test_bf16_few_tiles_of_long_contractions(T, d, f, E, k, kw):
    """Too few 256-row tiles for the chip: 64- or 128-row tiles in their place, most of them cut along K."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", [
    # 64-row tiles: single rows, K slices of the down-projection / of both input-gradient passes / of the up-projection
    (1, 264, 200, 4, 2, {}), (33, 72, 2056, 4, 2, {}), (40, 2056, 72, 5, 2, {}), (128, 1024, 64, 4, 1, {}),
    # 128-row tiles, an expert with two of them, dropped pairs
    (200, 136, 1096, 4, 2, {}), (220, 1032, 128, 4, 2, dict(bias=[2.0, 0, 0, 0])), (210, 320, 520, 4, 2, dict(cf=0.8, poison=True)),
    # 192-row tiles, groups on both sides of 192 rows
    (1120, 520, 392, 64, 8, {}), (1280, 512, 400, 64, 8, {}),
    # 256-row tiles with every form of the last k tile
    (1600, 520, 544, 64, 8, {}), (1700, 544, 576, 64, 8, {}),
    # few 256-row tiles: 128 or 64 rows in their place
    (600, 512, 176, 4, 2, {}), (700, 64, 1376, 3, 2, {}),
])
def test_bf16_row_tiles(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, **kw)


@pytest.mark.parametrize("nbytes", [None, 0, 300])
def test_a_workspace_that_is_too_small_is_replaced(nbytes):
    """The binding hands a workspace of its own to the calls, with the same results."""
    T, d, f, E, k = 70, 64, 96, 4, 2
    G = to_dev(synth.make_layer(T, d, f, E, dtype=F32, with_dY=True))
    def run(ws):
        r = B.btx_moe_route(G["x"], G["W_router"], k=k, workspace=ws)
        out, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r, workspace=ws)
        g = B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3, workspace=ws)
        return out, r.gates, g.dX, g.dW1, g.dW2
    expected = run(torch.empty(1 << 24, dtype=torch.uint8, device="cuda"))
    for a, b in zip(expected, run(None if nbytes is None else torch.empty(nbytes, dtype=torch.uint8, device="cuda"))):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T,d,f,E,k,dtype", [
    (16, 4096, 1024, 4, 2, BF16), (301, 1032, 4104, 4, 2, BF16), (33, 72, 2056, 4, 2, BF16), (40, 2056, 72, 5, 2, BF16),
    (900, 256, 2048, 4, 1, BF16), (210, 2056, 520, 4, 2, BF16), (260, 4104, 768, 16, 8, BF16), (2050, 1032, 8192, 2, 1, BF16),
    (64, 512, 1376, 8, 2, F32), (768, 512, 1376, 8, 2, F32), (1, 64, 2056, 3, 2, F32), (2003, 264, 1376, 4, 2, F32)])
def test_nothing_is_written_behind_the_workspace(T, d, f, E, k, dtype):
    """Workspaces of exactly the size that the queries return, products cut along K of every kind."""
    lib, code = B.load_library(), B.BTX_BF16 if dtype == BF16 else B.BTX_F32
    L = synth.make_layer(T, d, f, E, dtype=dtype, device="cuda", unit_rms=True, with_dY=True)
    r = B.btx_moe_route(L["x"], L["W_router"], None, None, k)
    behind = 128 << 20

    def workspace(nbytes):
        whole = torch.full((nbytes + behind,), 0xA5, dtype=torch.uint8, device="cuda")
        return whole[:nbytes], whole[nbytes:]
    ws, after = workspace(lib.btx_moe_ff_forward_workspace_bytes(T, d, f, E, k, code))
    out, h1, h3 = B.btx_moe_ff_forward(L["x"], L["W1"], L["W3"], L["W2"], r, workspace=ws)
    assert bool((after == 0xA5).all())
    ws, after = workspace(lib.btx_moe_ff_backward_workspace_bytes(T, d, f, E, k, code))
    B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3, workspace=ws)
    assert bool((after == 0xA5).all())


@pytest.mark.parametrize("T,d,f,E,k,kw", [
    # strips: no rows at all for some experts, one k tile, several k tiles (skewed), partial row panels and column tiles
    (3, 136, 264, 64, 2, {}), (64, 256, 192, 8, 2, {}), (100, 264, 136, 8, 4, dict(bias=[3.0] + [0.0] * 7)),
    (250, 512, 320, 16, 4, dict(cf=0.8, poison=True)), (256, 264, 1032, 4, 1, {}),
    # the same widths past the strips' limit of 64 rows per expert, whole lines and not
    (300, 256, 192, 4, 1, {}), (300, 264, 136, 4, 1, {}),
])
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_of_few_rows(T, d, f, E, k, kw, dW_dtype):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, **kw)


@pytest.mark.parametrize("T,d,f,E,k,bias", [
    (500, 264, 136, 8, 1, [6.0]), (512, 520, 264, 16, 2, [6.0, 6.0]),          # nearly everything on one expert, on two
    (800, 1032, 1032, 64, 2, [4.0, 3.5, 3.0, 3.0, 2.5]),                        # strips of several tiles, shorter for some
    (4000, 72, 136, 64, 1, [6.0]),
])
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_of_few_rows_with_overloaded_experts(T, d, f, E, k, bias, dW_dtype):
    """Up to 64 rows per expert on average, but far more on some: their strips are shared out over all workgroups."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, bias=bias + [0.0] * (E - len(bias)), poison=True)


@pytest.mark.parametrize("T,d,f,E,k,bias", [
    # one, two and most of the experts long; fewer strips than XCDs, shares that do not come out even, more strips than workgroups
    (400, 72, 72, 2, 1, [4.0]), (900, 264, 392, 7, 1, [0.0, 4.0]), (600, 1032, 264, 33, 2, [5.0, 0.0, 0.0, 5.0]), (1200, 264, 136, 5, 2, [3.0, 3.0, 3.0, 0.0, -60.0]),
    (700, 2056, 1096, 16, 1, [4.0, 0.0, 3.0]), (300, 520, 136, 64, 1, [7.0]),
])
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_of_long_experts_reach_every_tile(T, d, f, E, k, bias, dW_dtype):
    """The strips of experts with more rows than the average are dealt out first, to all XCDs: nothing is left as it was handed over."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, bias=bias + [0.0] * (E - len(bias)), poison=True)


@pytest.mark.parametrize("T,d,f,E,k,kw", [
    # one column tile and a little more of either operand, k tiles of 32 rows and their remainders, token rows of 1, 2, 3, 5 slots
    (256, 264, 136, 4, 1, {}), (257, 248, 128, 4, 2, {}), (303, 520, 264, 3, 3, {}), (161, 1032, 392, 7, 5, {}), (97, 128, 520, 1, 1, {}),
    # several k tiles on some experts, none on others; dropped pairs
    (900, 520, 264, 8, 2, dict(bias=[3.0] + [0.0] * 7, poison=True)), (700, 264, 520, 6, 3, dict(cf=0.8, poison=True)),
    # both sides of the limits: 360 rows, rows x width, and rows of few strips
    (720, 512, 520, 4, 2, {}), (722, 504, 520, 4, 2, {}), (2500, 520, 512, 2, 2, {}), (2560, 520, 512, 2, 2, {}),
    (720, 264, 5504, 2, 1, {}), (724, 264, 5504, 2, 1, {}), (1400, 72, 136, 4, 2, {}), (1404, 72, 136, 4, 2, {}), (1500, 256, 192, 8, 2, {}),
])
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_from_token_rows(T, d, f, E, k, kw, dW_dtype):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", DY_ROWS + DY_TRANSPOSED)
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_of_tiles_from_token_rows_of_dY(T, d, f, E, k, kw, dW_dtype):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, **kw)


@pytest.mark.parametrize("d", [64, 4096])          # rows transposed, and token rows as they lie
def test_bf16_an_infinity_in_the_last_row_of_dY_stays_in_its_column(d):
    """The last k tile's rows past the expert's last one repeat it: they must not turn its infinity into NaN."""
    T, f = 1001, 1400
    G = to_dev(synth.make_layer(T, d, f, 1, dtype=BF16, with_dY=True, unit_rms=True))
    r = B.btx_moe_route(G["x"], G["W_router"], k=1)
    _, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r)
    def dW2(dY):
        return B.btx_moe_ff_backward(dY, G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3).dW2[0].float()
    finite, broken = dW2(G["dY"]), G["dY"].clone()
    broken[-1, 17] = float("inf")
    got = dW2(broken)
    others = [c for c in range(d) if c != 17]
    assert torch.equal(got[:, others], finite[:, others])
    act = torch.nn.functional.silu(h1[-1].float()) * h3[-1].float()
    assert torch.equal(got[:, 17], torch.where(act > 0, torch.inf, -torch.inf))


def test_bf16_weight_gradients_from_token_rows_of_dY_past_2_gib():
    """Byte offsets of dY's rows from 2^31 on: as the same rows give in batches that stay below, fp32 sums of 500 thousand terms of random
    signs in two orders.  One expert, whose gate is 1."""
    T, d, f = 500_000, 4104, 72
    g = torch.Generator(device="cuda").manual_seed(8)
    x, dY = (torch.randn((T, d), generator=g, device="cuda", dtype=BF16) for _ in range(2))
    W1, W3 = (torch.randn((1, d, f), generator=g, device="cuda", dtype=BF16) * d ** -0.5 for _ in range(2))
    W2, Wr = torch.randn((1, f, d), generator=g, device="cuda", dtype=BF16) * f ** -0.5, torch.zeros((d, 1), device="cuda")

    def step(rows):
        r = B.btx_moe_route(x[rows], Wr, None, None, 1, B.BTX_ROUTE_SWITCH_TOP1)
        _, h1, h3 = B.btx_moe_ff_forward(x[rows], W1, W3, W2, r)
        b = B.btx_moe_ff_backward(dY[rows], x[rows], Wr, W1, W3, W2, r, h1, h3, B.BTX_ROUTE_SWITCH_TOP1, dW_dtype=F32)
        return [t[0].double() for t in (b.dW1, b.dW3, b.dW2)]

    whole, parts = step(slice(0, T)), [0.0] * 3
    for at in range(0, T, T // 4):
        parts = [a + b for a, b in zip(parts, step(slice(at, at + T // 4)))]
    for got, want in zip(whole, parts):
        assert float((got - want).norm() / want.norm()) < TOL[F32] / 4


@pytest.mark.parametrize("T,d,f,E,k,kw", ROW_PITCH)
def test_bf16_rows_of_experts_that_start_on_whole_lines(T, d, f, E, k, kw):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, poison=True, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", TRANSPOSED_ROWS)
@pytest.mark.parametrize("dW_dtype", [BF16, F32])
def test_bf16_weight_gradients_from_transposed_rows(T, d, f, E, k, kw, dW_dtype):
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=dW_dtype, **kw)


@pytest.mark.parametrize("T,d,f,E,k", [(90, 72, 72, 3, 2), (70, 120, 200, 2, 1), (100, 184, 184, 5, 2), (64, 200, 64, 2, 2), (77, 264, 8, 3, 1), (65, 320, 136, 2, 1),
                                       (130, 328, 192, 4, 2), (40, 376, 248, 4, 3), (33, 456, 256, 1, 1)])
def test_bf16_fp32_weight_gradients_of_few_rows_at_every_column_remainder(T, d, f, E, k):
    """fp32 strips: a lane holds 4 columns in each half of a 128-column piece; the last piece ends before, in and behind the halves."""
    run_layer_and_check(T, d, f, E, k, BF16, unit_rms=True, dW_dtype=F32, poison=True)


@pytest.mark.parametrize("T,d,E,k,kw", [
    # both sides of the limits of the two-launch routing: tokens, pairs, tokens x columns x experts
    (512, 64, 8, 8, {}), (513, 64, 8, 2, {}), (512, 72, 9, 8, dict(cf=0.8)), (456, 64, 9, 9, {}), (512, 1024, 64, 3, {}),
    (512, 1032, 64, 3, {}), (1, 4104, 5, 3, {}), (17, 2056, 3, 1, dict(mode=B.BTX_ROUTE_SWITCH_TOP1, cf=1.5)),
    (500, 64, 1, 1, dict(mode=B.BTX_ROUTE_SAMPLE_TOP1)), (499, 136, 33, 1, dict(mode=B.BTX_ROUTE_GUMBEL_TOP1)),
])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_routing_of_few_tokens(T, d, E, k, kw, dtype):
    run_layer_and_check(T, d, 64, E, k, dtype, unit_rms=True, backward=False, **kw)


@pytest.mark.parametrize("T,d,f,E,k,kw", [
    # 1, 2, 3 and 8 slots in registers (12: a finishing kernel adds them); an odd number of slices, dropped pairs
    (9, 264, 2056, 4, 1, {}), (20, 72, 2056, 5, 2, {}), (17, 264, 1544, 6, 3, dict(cf=0.8, poison=True)), (20, 264, 2056, 12, 12, {}),
    (5, 1032, 1096, 8, 8, {}),
])
@pytest.mark.parametrize("dtype", [BF16, F32])
def test_combine_adds_the_slices_of_the_down_projection(T, d, f, E, k, kw, dtype):
    run_layer_and_check(T, d, f, E, k, dtype, unit_rms=True, backward=False, **kw)


# 64-, 128-, 192- and 256-row tiles; the same, one expert with several of them
@pytest.mark.parametrize("T,k,bias", [(16, 2, 0.0), (160, 2, 0.0), (301, 2, 0.0), (420, 2, 0.0), (160, 1, 2.0), (320, 1, 2.0), (600, 1, 2.0), (900, 1, 2.0)])
def test_bf16_weights_streamed_past_the_caches_give_the_same_bits(T, k, bias):
    """1.1 GB of expert weights, read past the caches where their rows start on whole lines; shifted by 64 bytes they are not."""
    d, f, E = 4096, 11008, 4
    L = synth.make_layer(T, d, f, E, dtype=BF16, device="cuda", unit_rms=True, with_dY=True, router_bias=[bias, 0.0, 0.0, 0.0])
    r = B.btx_moe_route(L["x"], L["W_router"], L["b_router"], None, k)

    def shifted(W):
        return torch.empty(W.numel() + 64, dtype=W.dtype, device="cuda")[32:32 + W.numel()].view(W.shape).copy_(W)
    results = []
    for W1, W3, W2 in ((L["W1"], L["W3"], L["W2"]), tuple(shifted(L[n]) for n in ("W1", "W3", "W2"))):
        out, h1, h3 = B.btx_moe_ff_forward(L["x"], W1, W3, W2, r)
        g = B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], W1, W3, W2, r, h1, h3)
        results.append((out, h1, h3, g.dX, g.dW_router, g.dW1, g.dW3, g.dW2))
    assert all(torch.equal(a, b) for a, b in zip(*results))


@pytest.mark.parametrize("T,d,E,k,kw", [
    # one, two and four pairs a thread; all probabilities at once, in several pieces; 1024 tokens and one more
    (256, 64, 4, 4, {}), (257, 64, 4, 4, {}), (301, 64, 64, 2, {}), (64, 64, 17, 16, dict(cf=0.8)), (512, 72, 64, 8, dict(cf=1.25)),
    (1024, 64, 4, 4, {}), (1025, 64, 4, 2, {}), (1024, 2936, 4, 2, {}), (640, 72, 16, 6, {}), (641, 72, 16, 6, {}), (1000, 64, 1, 1, {}),
    (999, 72, 3, 1, dict(mode=B.BTX_ROUTE_SWITCH_TOP1, cf=0.5, bias=[2.0, 0.0, 0.0])),
])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_routing_by_one_workgroup(T, d, E, k, kw, dtype):
    run_layer_and_check(T, d, 64, E, k, dtype, unit_rms=True, backward=False, **kw)


@pytest.mark.parametrize("E", [2, 4, 8, 12])
def test_routing_takes_a_router_matrix_at_any_float(E):
    T, d, k = 50, 264, 2
    L = synth.make_layer(T, d, 64, E, dtype=BF16, device="cuda", unit_rms=True)
    shifted = torch.empty(d * E + 1, device="cuda")[1:].view(d, E).copy_(L["W_router"])
    a, b = (B.btx_moe_route(L["x"], W, None, None, k, B.BTX_ROUTE_TOPK_RENORM, B.BTX_LB_TOKEN_FRAC, 0.01)
            for W in (L["W_router"], shifted))
    for x, y in zip(vars(a).values(), vars(b).values()):
        if torch.is_tensor(x):
            assert torch.equal(x, y)


@pytest.mark.parametrize("T", [300, 1500])               # two launches, four launches
@pytest.mark.parametrize("E,k", [(4, 2), (12, 5)])
@pytest.mark.parametrize("broken", ["row", "expert"])
def test_routing_of_nan_logits_fills_every_slot(T, E, k, broken):
    """A row (or one expert's column of W_router) that holds NaN: its gates mean nothing, but k different experts are chosen,
    whatever the output buffers held before, and the other rows are routed as ever."""
    L = to_dev(synth.make_layer(T, 64, 64, E, dtype=F32))
    clean = B.btx_moe_route(L["x"], L["W_router"], None, None, k)
    if broken == "row":
        L["x"][7] = float("nan")
    else:
        L["W_router"][:, 1] = float("nan")
    runs = []
    for fill in (1, 3):
        r = B.alloc_routing(T, E, k, "cuda")
        for t in vars(r).values():
            t.fill_(fill)
        B.btx_moe_route(L["x"], L["W_router"], None, None, k, out=r)
        runs.append(r)
    for a, b in zip(vars(runs[0]).values(), vars(runs[1]).values()):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    idx = runs[0].topk_idx.long()
    assert bool(((idx >= 0) & (idx < E)).all()) and bool((idx.sort(dim=1).values.diff(dim=1) > 0).all())
    assert torch.equal(runs[0].counts.long(), torch.bincount(idx.flatten(), minlength=E))
    assert torch.equal(runs[0].perm.sort().values, torch.arange(T * k, dtype=torch.int32, device="cuda"))
    assert torch.equal(runs[0].perm[runs[0].inv_pos.flatten().long()], torch.arange(T * k, dtype=torch.int32, device="cuda"))
    if broken == "row":
        rest = torch.arange(T, device="cuda") != 7
        assert torch.equal(idx[rest], clean.topk_idx.long()[rest]) and torch.equal(runs[0].gates[rest], clean.gates[rest])


def test_bf16_unrelated_experts_meet_the_plain_bar_on_router_gradients():
    """With experts that share nothing the gate Jacobian has no cancellation and
    dW_router / db_router must meet 2e-2 without any amplification factor."""
    run_layer_and_check(1024, 256, 384, 4, 2, BF16, unit_rms=True, expert_spread=3.0)


@pytest.mark.parametrize("T,d,f", [(300, 128, 256), (150, 96, 416)])
def test_bf16_fp32_weight_gradients(T, d, f):
    run_layer_and_check(T, d, f, 4, 2, BF16, unit_rms=True, dW_dtype=F32)


def test_bf16_switch_imbalanced():
    run_layer_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[2.0, 0, 0, 0], unit_rms=True)


def test_bf16_sample_top1_imbalanced():
    run_layer_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_SAMPLE_TOP1, bias=[2.0, 0, 0, 0], unit_rms=True)


def test_bf16_gumbel_sample_top1():
    run_layer_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_GUMBEL_TOP1, unit_rms=True, tau=0.5)


def test_bf16_switch_with_capacity_factor():
    """Switch routing at capacity factor 1.5 with a router that overloads expert 0 (Sec. 4.3)."""
    G, r, out, g = run_layer_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[2.0, 0, 0, 0],
                                       unit_rms=True, cf=1.5)
    assert int((r.inv_pos < 0).sum()) > 0 and int(r.offsets[1]) == 338   # ceil(1.5 * 900 / 4)


def test_capacity_limit_follows_the_float_that_was_passed():
    """cf = 0.8 reaches the library as the float32 nearest to 0.8, which lies above it: at T/E = 260 the
    limit is 209 rows, not 208; the oracle is given the same number."""
    G, r, out, g = run_layer_and_check(1040, 128, 96, 4, 1, F32, mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[1.5, 0, 0, 0],
                                       cf=0.8)
    assert int(r.offsets[1]) == 209


def test_bf16_top2_with_capacity_factor():
    run_layer_and_check(1500, 512, 1376, 8, 4, BF16, unit_rms=True, cf=0.75, bias=[1.0, 0.5, 0, 0, 0, 0, -0.5, -1.0])


@pytest.mark.parametrize("case", ["switch-cf", "top2-cf", "many-experts-cf", "top2-dropless", "ragged-dropless",
                                  "fp32-cf", "fp32-dw-cf"])
def test_nothing_depends_on_unwritten_workspace(case):
    """Workspace, saved activations and outputs are handed over with every byte 0xFF (NaN patterns).
    With a capacity limit the grouped rows behind the last kept one are never written by the
    backward stages, and the weight-gradient products pad every expert's rows to whole k tiles:
    whatever those padded k rows read is multiplied by zeros and must therefore be finite."""
    kw = dict(unit_rms=True, poison=True)
    if case == "switch-cf":
        run_layer_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[2.0, 0, 0, 0], cf=1.5, **kw)
    elif case == "top2-cf":
        run_layer_and_check(1500, 512, 1376, 8, 4, BF16, cf=0.75, bias=[1.0, 0.5, 0, 0, 0, 0, -0.5, -1.0], **kw)
    elif case == "many-experts-cf":
        run_layer_and_check(700, 96, 160, 24, 3, BF16, cf=0.5, **kw)
    elif case == "top2-dropless":
        run_layer_and_check(512, 256, 384, 4, 2, BF16, **kw)
    elif case == "ragged-dropless":
        run_layer_and_check(333, 320, 96, 5, 3, BF16, bias=[0, -60.0, 0, 0, 0], **kw)
    elif case == "fp32-cf":
        run_layer_and_check(301, 72, 88, 5, 3, F32, cf=0.6, poison=True)
    else:
        run_layer_and_check(300, 128, 256, 4, 2, BF16, dW_dtype=F32, cf=0.7, **kw)


@pytest.mark.parametrize("dW_dtype", [BF16, F32])
@pytest.mark.parametrize("T,d,f,E,k", [(1, 64, 64, 2, 1), (3, 64, 72, 2, 1), (40, 72, 64, 3, 2), (33, 136, 264, 9, 2), (130, 264, 72, 64, 8), (70, 8, 2056, 4, 2)])
def test_strips_of_all_weight_gradients_in_one_launch(T, d, f, E, k, dW_dtype):
    """Fewer tiles than XCDs and more, either product's stores past the caches, both and neither."""
    run_layer_and_check(T, d, f, E, k, BF16, dW_dtype=dW_dtype, poison=True)


def test_bf16_expert_without_tokens():
    run_layer_and_check(300, 128, 256, 4, 2, BF16, bias=[0, -60.0, 0, 0], unit_rms=True)


# ------------------------------------------------- the sublayer in its block
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,d,E,k", [(3, 72, 8, 3), (64, 520, 4, 2), (65, 2056, 5, 2), (128, 1032, 9, 4), (129, 64, 33, 5), (257, 1544, 64, 2),
                                     (4100, 136, 24, 12)])
def test_router_gradients_and_dX_in_one_launch(T, d, E, k, dtype):
    """One and several chunks of tokens, column blocks that end early, experts that take turns in LDS, more slots than eight."""
    run_layer_and_check(T, d, 72, E, k, dtype, unit_rms=True, poison=True)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("E,k", [(3, 2), (8, 1)])
def test_router_gradients_of_large_batches(E, k, dtype):
    """The last 16 tokens of a wavefront and the last chunk of 64 have one."""
    run_layer_and_check(32705, 8, 8, E, k, dtype, unit_rms=True, poison=True)


@pytest.mark.parametrize("T,d,E,k", [(5400, 1032, 64, 2), (8000, 1544, 17, 1)])
def test_router_gradients_of_many_experts_in_a_launch_of_their_own(T, d, E, k):
    """The sizes for which the partial sums do not run beside dX: passes of 16 experts, the last one of 1 and of 16."""
    run_layer_and_check(T, d, 8, E, k, BF16, unit_rms=True, poison=True)


@pytest.mark.parametrize("T,d,f,E,k,dtype", [
    (300, 64, 176, 4, 2, F32),          # fp32, ragged last token block
    (77, 2056, 64, 3, 1, F32),          # d not a multiple of the 2048-column thread stride, E < 4
    (1000, 512, 1376, 8, 2, BF16),      # 250 rows per expert
    (515, 4096, 256, 4, 2, BF16),       # the benchmark's d
    (130, 4608, 128, 16, 4, BF16),      # E > 8: several expert passes over the rows; d > 4096
])
def test_block_rmsnorm_route_forward_backward(T, d, f, E, k, dtype):
    run_block_and_check(T, d, f, E, k, dtype)


@pytest.mark.parametrize("T,d,E,k,dtype", ROUTE_AHEAD)
def test_block_rmsnorm_route_of_few_wide_rows(T, d, E, k, dtype):
    run_block_and_check(T, d, 64, E, k, F32 if dtype == B.BTX_F32 else BF16)


@pytest.mark.parametrize("T,d,E,k,dtype", [
    # few experts go to the two launches up to 1024 tokens, to 16 or 4 wavefronts for 16 tokens above (see ROUTE_MANY); ragged last blocks
    (601, 136, 3, 2, BF16), (523, 1032, 40, 4, BF16), (601, 136, 40, 3, F32), (530, 1032, 5, 2, F32), (515, 8200, 3, 2, F32),
    (4203, 72, 33, 2, BF16), (4203, 72, 9, 2, F32), (4203, 4104, 3, 1, F32), (8190, 72, 5, 3, BF16),
])
def test_block_rmsnorm_route_wavefronts(T, d, E, k, dtype):
    run_block_and_check(T, d, 64, E, k, dtype)


@pytest.mark.parametrize("T,d,E,k,dtype", [(601, 136, 3, 2, BF16), (4203, 1032, 7, 2, F32), (4203, 136, 7, 2, BF16), (600, 8200, 2, 1, F32),
                                           (4203, 72, 12, 3, F32), (4203, 2056, 40, 2, BF16), (8190, 72, 17, 2, BF16)])
def test_routing_wavefronts(T, d, E, k, dtype):
    """Without the normalisation: the vector unit up to 8 experts, the matrix cores beyond."""
    run_layer_and_check(T, d, 64, E, k, dtype, unit_rms=True, backward=False)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,d,E", [(700, 8, 9), (700, 40, 16), (4203, 48, 17), (700, 56, 31), (4203, 64, 32), (700, 136, 33), (8200, 144, 48), (700, 264, 49),
                                   (4203, 1032, 63), (700, 1048, 64)])
def test_routing_reads_every_column_of_every_expert(T, d, E, dtype):
    """More than 8 experts: W_router in pieces of 32 columns (the last of 8, 16 or 24) and 16 experts (the last of 1, 15 or 16)."""
    run_layer_and_check(T, d, 8, E, 2, dtype, unit_rms=True, backward=False, poison=True)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,d,E", [(4203, 40, 33), (4203, 264, 33), (8200, 264, 24), (4203, 392, 49), (8200, 520, 9), (4203, 648, 40), (700, 904, 64),
                                   (4203, 4104, 12), (4203, 4200, 20)])
def test_routing_trips_that_are_no_whole_rounds(T, d, E, dtype):
    """More than 8 experts: no trip, one to six and more for each wavefront, of which two or three are on their way at a time."""
    run_layer_and_check(T, d, 8, E, 2, dtype, unit_rms=True, backward=False, poison=True)


@pytest.mark.parametrize("case,taken", ROUTE_MANY)
def test_routing_of_many_tokens(case, taken):
    """Every number of experts in a pass and of wavefronts that share 16 tokens, above the sizes that two launches take."""
    T, d, E, k, code, norm = case
    dtype = BF16 if code == B.BTX_BF16 else F32
    if norm:
        run_block_and_check(T, d, 64, E, k, dtype)
    else:
        run_layer_and_check(T, d, 64, E, k, dtype, unit_rms=True, backward=False)


def test_block_rmsnorm_with_switch_routing_and_capacity():
    run_block_and_check(900, 256, 256, 4, 1, BF16, mode=B.BTX_ROUTE_SWITCH_TOP1, bias=[2.0, 0, 0, 0], cf=1.5)


def test_block_rmsnorm_route_matches_plain_route_on_the_normalised_rows():
    """The fused kernel must route exactly as btx_moe_route does when handed the rows it wrote."""
    L = synth.make_layer(700, 512, 64, 8, dtype=BF16)
    h = (L["x"].float() * 3.0).to(BF16).cuda()
    gain = torch.linspace(0.5, 1.5, 512).cuda()
    Wr = L["W_router"].cuda()
    r1, xn, _ = B.btx_moe_norm_route(h, gain, 1e-5, Wr, k=2, lb_alpha=0.01)
    r2 = B.btx_moe_route(xn, Wr, k=2, lb_alpha=0.01)
    for name in ("topk_idx", "gates", "probs", "counts", "offsets", "perm", "inv_pos", "gate_sum", "prob_sum", "lb_loss"):
        assert torch.equal(getattr(r1, name), getattr(r2, name)), name


@pytest.mark.parametrize("T,d,E,dtype", [(600, 4096, 4, BF16), (3001, 1032, 7, BF16), (4201, 2048, 8, BF16), (700, 512, 8, F32), (4201, 512, 3, F32),
                                         (530, 8200, 2, F32), (1024, 4096, 4, BF16), (640, 4096, 8, BF16), (1024, 8200, 4, F32), (520, 4104, 7, F32),
                                         (1030, 8200, 2, F32), (1100, 1032, 3, BF16), (1035, 4096, 4, BF16)])
def test_block_rmsnorm_route_gives_the_same_bits_with_other_wavefronts(T, d, E, dtype):
    """Sizes where the fused kernel and btx_moe_route split the tokens of a block over different numbers of wavefronts, and sizes
    between those that few tokens' kernels take and those that they do not."""
    h = (synth.make_layer(T, d, 64, E, dtype=dtype)["x"].float() * 3.0).to(dtype).cuda()
    gain = torch.linspace(0.5, 1.5, d).cuda()
    Wr = 0.02 * torch.randn((d, E), generator=torch.Generator().manual_seed(E)).cuda()
    r1, xn, _ = B.btx_moe_norm_route(h, gain, 1e-5, Wr, k=2, lb_alpha=0.01)
    r2 = B.btx_moe_route(xn, Wr, k=2, lb_alpha=0.01)
    for a, b in zip(vars(r1).values(), vars(r2).values()):
        assert torch.equal(a, b)


# ---------------------------------------------------------------------- merge
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 7])
def test_merge_of_identical_copies_is_the_identity(dtype, n):
    t = (torch.randn(100003, generator=torch.Generator().manual_seed(1)) * 3).to(dtype).cuda()
    out = B.btx_merge_average([t.clone() for _ in range(n)])
    assert torch.equal(out, t)


@pytest.mark.parametrize("n", [2, 3, 4, 5])
def test_merge_bf16_matches_oracle_bit_exactly(n):
    sets = synth.make_merge_set([(257, 129)], n, dtype=BF16)[0]
    want = O.round_to_bf16(O.merge_average([to_np(t) for t in sets]))
    got = B.btx_merge_average([t.cuda() for t in sets])
    assert np.array_equal(got.float().cpu().numpy(), want)


def test_merge_fp32_matches_oracle():
    sets = synth.make_merge_set([(1000, 37)], 3, dtype=F32)[0]
    want = O.merge_average([to_np(t) for t in sets])
    got = B.btx_merge_average([t.cuda() for t in sets])
    np.testing.assert_allclose(got.cpu().numpy(), want, rtol=3e-7, atol=0)


def test_merge_in_place():
    sets = [t.cuda() for t in synth.make_merge_set([(64, 64)], 4, dtype=BF16)[0]]
    want = B.btx_merge_average(sets)
    B.btx_merge_average(sets, out=sets[0])
    assert torch.equal(sets[0], want)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("weights", [[0.5, 0.25, 0.25], [0.7, 0.1, 0.15, 0.05], [1.0], [2.0, -1.0], [0.3, 0.3, 0.3, 0.3, 0.3]])
def test_weighted_merge_matches_the_oracle_bit_for_bit(dtype, weights):
    """fp64 accumulation in input order on both sides (every product is exact in fp64) and one
    rounding to the storage type: the results must be identical, ragged tail included."""
    sets = synth.make_merge_set([(257, 131)], len(weights), dtype=dtype)[0]
    w32 = [float(np.float32(w)) for w in weights]            # the ABI takes float weights
    acc = O.merge_weighted([to_np(t) for t in sets], w32)
    want = O.round_to_bf16(acc) if dtype == BF16 else acc.astype(np.float32)
    got = B.btx_merge_weighted([t.cuda() for t in sets], weights)
    assert np.array_equal(got.float().cpu().numpy(), want)


def test_weighted_merge_special_cases():
    sets = [t.cuda() for t in synth.make_merge_set([(300, 77)], 4, dtype=BF16)[0]]
    # a one-hot weight vector selects that model, bit for bit
    assert torch.equal(B.btx_merge_weighted(sets, [0.0, 0.0, 1.0, 0.0]), sets[2])
    # weights 1/4 are exact in binary: the weighted merge then is the plain average
    assert torch.equal(B.btx_merge_weighted(sets, [0.25] * 4), B.btx_merge_average(sets))
    # in place
    want = B.btx_merge_weighted(sets, [0.4, 0.3, 0.2, 0.1])
    B.btx_merge_weighted(sets, [0.4, 0.3, 0.2, 0.1], out=sets[0])
    assert torch.equal(sets[0], want)


# ------------------------------------------------------------- split / blend
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,d,f,C", [(4, 64, 96, 3), (2, 40, 36, 2), (3, 24, 30, 5), (1, 16, 64, 8)])
def test_split_and_blend_match_the_oracle_bit_for_bit(dtype, N, d, f, C):
    """Pure re-indexing: every element must arrive unchanged, also where the chunk width is
    not a whole number of 16-byte units (scalar copy path)."""
    L = synth.make_layer(8, d, f * (N if f % N else 1), N, dtype=dtype)
    G = to_dev(L)
    W1, W3, W2 = G["W1"], G["W3"], G["W2"]
    n1, n3, n2 = experts_np(L["W1"]), experts_np(L["W3"]), experts_np(L["W2"])
    if W1.shape[2] % C == 0:
        g1, g3, g2 = B.split_experts(W1, W3, W2, C)
        o1, o3, o2 = O.split_experts(n1, n3, n2, C)
        for g, o in ((g1, o1), (g3, o3), (g2, o2)):
            assert g.shape[0] == N * C
            assert np.array_equal(to_np(g), np.stack(o))
    g1, g3, g2 = B.blend_experts(W1, W3, W2)
    o1, o3, o2 = O.blend_experts(n1, n3, n2)
    for g, o in ((g1, o1), (g3, o3), (g2, o2)):
        assert np.array_equal(to_np(g), np.stack(o))
    # dealing out twice restores the input
    b1, b3, b2 = B.blend_experts(g1, g3, g2)
    assert torch.equal(b1, W1) and torch.equal(b3, W3) and torch.equal(b2, W2)


def test_two_layers_on_two_streams_do_not_disturb_each_other():
    """Nothing in the library is shared between calls but what the caller passes: two layers of different
    shapes enqueued alternately on two streams (default priority) give, bit for bit, what each gives alone."""
    cases = [(700, 256, 384, 4, 2), (512, 128, 2048, 3, 1)]
    layers, alone = [], []
    for (T, d, f, E, k) in cases:
        G = to_dev(synth.make_layer(T, d, f, E, dtype=BF16, unit_rms=True, with_dY=True, seed=synth.BASE_SEED + d))
        mode = B.BTX_ROUTE_TOPK_RENORM if k > 1 else B.BTX_ROUTE_SWITCH_TOP1
        r = B.btx_moe_route(G["x"], G["W_router"], None, None, k, mode, lb_alpha=0.01)
        out, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r)
        g = B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3, mode,
                                  lb_alpha=0.01, lb_grad_scale=1.0)
        layers.append((G, k, mode))
        alone.append((r, out, g))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    both = [None, None]
    for rep in range(3):
        for i, (G, k, mode) in enumerate(layers):
            with torch.cuda.stream(streams[i]):
                r = B.btx_moe_route(G["x"], G["W_router"], None, None, k, mode, lb_alpha=0.01)
                out, h1, h3 = B.btx_moe_ff_forward(G["x"], G["W1"], G["W3"], G["W2"], r)
                g = B.btx_moe_ff_backward(G["dY"], G["x"], G["W_router"], G["W1"], G["W3"], G["W2"], r, h1, h3, mode,
                                          lb_alpha=0.01, lb_grad_scale=1.0)
                both[i] = (r, out, g)
    torch.cuda.synchronize()
    for (r0, out0, g0), (r1, out1, g1) in zip(alone, both):
        assert torch.equal(r0.perm, r1.perm) and torch.equal(out0, out1) and torch.equal(g0.dX, g1.dX)
        assert torch.equal(g0.dW1, g1.dW1) and torch.equal(g0.dW2, g1.dW2) and torch.equal(g0.dW_router, g1.dW_router)


def test_layer_step_replays_from_a_hip_graph():
    """The three entry points only enqueue kernels on the given stream (no allocation, no
    synchronisation, no memset nodes), so a whole step can be captured once and replayed.
    Every replay, with eager work in between, must reproduce the eager results bit for bit."""
    T, d, f, E, k = 700, 256, 384, 4, 2
    L = to_dev(synth.make_layer(T, d, f, E, dtype=BF16, unit_rms=True, with_dY=True))
    lib = B.load_library()
    routing = B.alloc_routing(T, E, k, "cuda")
    out = torch.empty_like(L["x"])
    saved = (torch.empty((T * k, f), dtype=BF16, device="cuda"), torch.empty((T * k, f), dtype=BF16, device="cuda"))
    grads = B.Grads(torch.empty_like(L["x"]), torch.empty((d, E), device="cuda"), torch.empty(E, device="cuda"),
                    torch.empty_like(L["W1"]), torch.empty_like(L["W3"]), torch.empty_like(L["W2"]))
    ws = torch.empty(max(lib.btx_moe_route_workspace_bytes(T, d, E, k),
                         lib.btx_moe_ff_forward_workspace_bytes(T, d, f, E, k, B.BTX_BF16),
                         lib.btx_moe_ff_backward_workspace_bytes(T, d, f, E, k, B.BTX_BF16)), dtype=torch.uint8,
                     device="cuda")

    def step():
        B.btx_moe_route(L["x"], L["W_router"], None, None, k, lb_alpha=0.01, out=routing, workspace=ws)
        B.btx_moe_ff_forward(L["x"], L["W1"], L["W3"], L["W2"], routing, out=out, saved=saved, workspace=ws)
        B.btx_moe_ff_backward(L["dY"], L["x"], L["W_router"], L["W1"], L["W3"], L["W2"], routing, saved[0], saved[1],
                              lb_alpha=0.01, lb_grad_scale=1.0, out=grads, workspace=ws)

    step()                                   # eager reference (also sets the kernels' LDS attributes)
    torch.cuda.synchronize()
    want = [t.clone() for t in (out, grads.dX, grads.dW_router, grads.dW1, grads.dW2, routing.perm)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for t in (out, grads.dX, grads.dW_router, grads.dW1, grads.dW2):
            t.zero_()                        # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip((out, grads.dX, grads.dW_router, grads.dW1, grads.dW2, routing.perm), want):
            assert torch.equal(got, ref)


def test_block_step_replays_from_a_hip_graph():
    """The same for the sublayer inside its block: norm + route, forward with the residual,
    backward, normalisation backward in place on dX."""
    T, d, f, E, k = 600, 256, 384, 4, 2
    L = to_dev(synth.make_layer(T, d, f, E, dtype=BF16, with_dY=True))
    h = (L["x"].float() * 2.5).to(BF16)
    gain = torch.linspace(0.8, 1.2, d, device="cuda")
    lib = B.load_library()
    routing = B.alloc_routing(T, E, k, "cuda")
    xn, rstd, out = torch.empty_like(h), torch.empty(T, device="cuda"), torch.empty_like(h)
    dgain = torch.empty(d, device="cuda")
    saved = (torch.empty((T * k, f), dtype=BF16, device="cuda"), torch.empty((T * k, f), dtype=BF16, device="cuda"))
    grads = B.Grads(torch.empty_like(h), torch.empty((d, E), device="cuda"), torch.empty(E, device="cuda"),
                    torch.empty_like(L["W1"]), torch.empty_like(L["W3"]), torch.empty_like(L["W2"]))
    ws = torch.empty(max(lib.btx_moe_route_workspace_bytes(T, d, E, k),
                         lib.btx_moe_ff_forward_workspace_bytes(T, d, f, E, k, B.BTX_BF16),
                         lib.btx_moe_ff_backward_workspace_bytes(T, d, f, E, k, B.BTX_BF16),
                         lib.btx_rmsnorm_backward_workspace_bytes(T, d)), dtype=torch.uint8, device="cuda")

    def step():
        B.btx_moe_norm_route(h, gain, 1e-5, L["W_router"], None, None, k, lb_alpha=0.01, out=routing, workspace=ws,
                             xn=xn, rstd=rstd)
        B.btx_moe_ff_forward(xn, L["W1"], L["W3"], L["W2"], routing, out=out, saved=saved, workspace=ws, residual=h)
        B.btx_moe_ff_backward(L["dY"], xn, L["W_router"], L["W1"], L["W3"], L["W2"], routing, saved[0], saved[1],
                              lb_alpha=0.01, lb_grad_scale=1.0, out=grads, workspace=ws)
        B.btx_rmsnorm_backward(grads.dX, h, gain, rstd, dres=L["dY"], dH=grads.dX, workspace=ws, dgain=dgain)

    step()
    torch.cuda.synchronize()
    watched = (xn, out, grads.dX, dgain, grads.dW3, routing.inv_pos)
    want = [t.clone() for t in watched]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for t in (xn, out, grads.dX, dgain, grads.dW3):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip(watched, want):
            assert torch.equal(got, ref)


# -------------------------------------------------------------------- AdamW
@pytest.mark.parametrize("gdtype", [F32, BF16])
@pytest.mark.parametrize("n,beta2", [(4096 * 33 + 3, 0.95), (5, 0.95), (1 << 20, 0.95), (65537, 0.999)])
def test_adamw_steps_follow_the_oracle(gdtype, n, beta2):
    """The hyper-parameters reach the library as C floats; the oracle is given the same numbers
    (1 - beta2 differs by 1.3e-5 between 0.999 and the float nearest to it)."""
    lr, beta1, beta2, eps, wd = (as_passed(v) for v in (1e-4, 0.9, beta2, 1e-8, 0.1))
    g = torch.Generator().manual_seed(n)
    p = torch.randn(n, generator=g) * 0.02
    m = torch.zeros(n)
    v = torch.zeros(n)
    P, M, V = p.cuda(), m.cuda(), v.cuda()
    low = torch.empty(n, dtype=BF16, device="cuda")
    po, mo, vo = p.double().numpy(), m.double().numpy(), v.double().numpy()
    for step in range(1, 4):
        grad = (torch.randn(n, generator=g) * 1e-3).to(gdtype)
        B.btx_adamw_step(P, M, V, grad.cuda(), step, lr, beta1, beta2, eps, wd, lowp=low)
        po, mo, vo = O.adamw_step(po, grad.double().numpy(), mo, vo, step, lr, beta1, beta2, eps, wd)
    # the update itself (weights move by ~1e-4 per step): compared as a difference from the start
    start = p.double().numpy()
    assert_close(P.cpu().double().numpy() - start, po - start, 1e-4, "update")
    assert_close(M.cpu().numpy(), mo, 1e-5, "m")
    assert_close(V.cpu().numpy(), vo, 1e-5, "v")
    # working copy: the fp32 result rounded once
    assert torch.equal(low, P.to(BF16))


@pytest.mark.parametrize("n", [11184810, 11184813])     # both sides of 128 MB of P, M and V; no multiple of 4
def test_adamw_past_the_caches_gives_the_same_numbers(n):
    """The update is elementwise: a tensor must come out as its pieces do."""
    g = torch.Generator(device="cuda").manual_seed(n)
    P, M = (torch.randn(n, generator=g, device="cuda") for _ in range(2))
    V = torch.rand(n, generator=g, device="cuda")
    grad = torch.randn(n, generator=g, device="cuda").to(BF16)
    whole, low = [t.clone() for t in (P, M, V)], torch.empty(n, dtype=BF16, device="cuda")
    B.btx_adamw_step(*whole, grad, 3, 1e-3, weight_decay=0.1, lowp=low)
    for lo in range(0, n, 4000000):
        piece = [t[lo:lo + 4000000].clone() for t in (P, M, V, grad)]
        low_p = torch.empty_like(piece[3])
        B.btx_adamw_step(*piece, 3, 1e-3, weight_decay=0.1, lowp=low_p)
        for got, want in zip([t[lo:lo + 4000000] for t in (*whole, low)], (*piece[:3], low_p)):
            assert torch.equal(got, want)
