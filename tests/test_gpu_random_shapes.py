"""Seeded random configurations of the whole layer (route, forward, backward) against the oracle:
both storage types, every routing mode, both forms of the load-balancing loss, capacity limits,
router biases, 1 to 64 experts, widths on and off the grid of 32 (in bf16 all of them on 64- and 128-row
tiles), poisoned workspaces.  The same generator with other seeds found the cases that tests elsewhere now
pin by name (wide experts off that grid, the capacity limit at an exact product, gradients whose sum over
the tokens cancels)."""
import numpy as np
import pytest
import torch

from paper_2403_07816_amd import binding as B
from paper_2403_07816_amd import synth

from helpers import run_layer_and_check

pytestmark = pytest.mark.gpu


def random_case(rng):
    dtype = torch.bfloat16 if rng.random() < 0.6 else torch.float32
    E = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 31, 32, 33, 48, 64]))
    mode = int(rng.choice([B.BTX_ROUTE_TOPK_RENORM, B.BTX_ROUTE_TOPK_RENORM, B.BTX_ROUTE_SWITCH_TOP1,
                           B.BTX_ROUTE_SAMPLE_TOP1, B.BTX_ROUTE_GUMBEL_TOP1]))
    k = int(rng.integers(1, min(E, 8) + 1)) if mode == B.BTX_ROUTE_TOPK_RENORM else 1
    step = 32 if (dtype == torch.bfloat16 and rng.random() < 0.8) else 8
    d = step * int(rng.integers(max(1, 64 // step), 400 // step))
    f = step * int(rng.integers(max(1, 64 // step), 500 // step))
    T = int(rng.integers(1, 900))
    kw = dict(mode=mode, alpha=float(rng.choice([0.0, 0.01, 0.5])), lam=float(rng.choice([0.0, 1.0])),
              tau=float(rng.choice([0.5, 1.0, 2.0])), lb_mode=int(rng.choice([B.BTX_LB_TOKEN_FRAC, B.BTX_LB_GATE_MEAN])))
    if kw["lb_mode"] == B.BTX_LB_GATE_MEAN and rng.random() < 0.5:
        kw["flags"] = B.BTX_FLAG_LB_GRAD_THROUGH_U
    if rng.random() < 0.3:
        kw["cf"] = float(rng.choice([0.5, 0.8, 1.0, 1.25, 1.5]))
    if rng.random() < 0.4:
        kw["bias"] = [float(v) for v in rng.normal(0, 1.0, E)]
    if dtype == torch.bfloat16:
        kw["unit_rms"] = True
        if rng.random() < 0.3:
            kw["dW_dtype"] = torch.float32
    kw["poison"] = bool(rng.random() < 0.5)
    return (T, d, f, E, k, dtype), kw


@pytest.mark.parametrize("seed", [101, 102, 103])
def test_random_layers_match_the_oracle(seed):
    rng = np.random.default_rng(seed)
    for i in range(25):
        args, kw = random_case(rng)
        print(f"seed {seed} case {i}: T,d,f,E,k,dtype = {args} {kw}", flush=True)
        run_layer_and_check(*args, seed=synth.BASE_SEED + 1000 * seed + i, **kw)
