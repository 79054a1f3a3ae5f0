"""The gate on the matrix cores at the sizes where its tilings can go wrong: ragged token tiles, the edges between the
four-, sixteen- and thirty-two-token tiles, expert counts that are no multiple of a lane's share, short last feature blocks,
empty partial sums, and logits in the subnormal range.  Routing is compared bit for bit, gate scales at rtol 1e-5 (expf)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,act,x_scale", [
    (1, 8, 2, 2, "f16", 1.0), (15, 40, 16, 2, "f16", 1.0), (17, 1032, 17, 2, "f16", 1.0), (16, 512, 31, 1, "bf16", 1.0),
    (3, 520, 33, 2, "f16", 1.0), (5, 1160, 64, 1, "bf16", 1.0), (1024, 136, 40, 2, "f16", 1.0), (1025, 136, 40, 2, "f16", 1.0),
    (1030, 264, 63, 2, "bf16", 1.0), (31, 776, 66, 2, "f16", 1.0), (49, 1096, 128, 2, "bf16", 1.0),
    (18, 904, 129, 1, "f16", 1.0), (33, 2048, 250, 2, "f16", 1.0), (16, 1024, 256, 2, "bf16", 1.0),
    (8160, 128, 32, 2, "f16", 1.0), (8161, 72, 32, 2, "f16", 1.0), (8191, 200, 64, 1, "bf16", 1.0), (8193, 64, 96, 2, "f16", 1.0),
    (40, 1024, 64, 2, "bf16", 2.0 ** -118), (40, 1024, 32, 2, "bf16", 2.0 ** -118)])
def test_gate_tile_edges_bit_exact(T, d, E, k, act, x_scale):
    print(f"gate tiles T={T} d={d} E={E} k={k} {act} x scaled by {x_scale}", flush=True)
    rng = np.random.default_rng(T + d + E)
    tdt = torch.float16 if act == "f16" else torch.bfloat16
    x = to_dev((rng.standard_normal((T, d)) * x_scale).astype(np.float32), tdt)
    wg = to_dev((rng.standard_normal((d, E)) * (0.02 if x_scale == 1.0 else 2.0 ** -16)).astype(np.float32), tdt)
    bias = rng.uniform(-0.2, 0.2, E).astype(np.float32) if T % 2 and x_scale == 1.0 else None
    oi, osc = oracle.gate(x.float().cpu().numpy(), wg.float().cpu().numpy(), bias, k, True)
    gi, gs = B.moe_gate_topk(x, wg, None if bias is None else to_dev(bias, torch.float32), k, True)
    torch.cuda.synchronize()
    assert np.array_equal(gi.cpu().numpy(), oi)
    assert np.allclose(gs.cpu().numpy(), osc, rtol=1e-5, atol=1e-9)
