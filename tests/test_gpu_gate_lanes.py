"""The gate's forms for few tokens: a block per token or two with 65 to 128 experts, and the wide loads of 33 to 64."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TORCH_DT, to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E", [(1, 8, 66), (5, 136, 126), (256, 640, 128), (257, 1032, 128), (511, 520, 100), (512, 2048, 96), (513, 64, 128),
                                   (3, 200, 36), (7, 1032, 64), (1024, 72, 60)])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_gate_few_tokens_bit_exact(T, d, E, act):
    print(f"gate T={T} d={d} E={E} {act}", flush=True)
    rng = np.random.default_rng(T + d + E)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), TORCH_DT[act])
    wg = to_dev((rng.standard_normal((d, E)) * 0.05).astype(np.float32), TORCH_DT[act])
    bias = (rng.standard_normal(E) * 0.05).astype(np.float32)
    for k in (1, 2):
        oi, osc = oracle.gate(x.float().cpu().numpy(), wg.float().cpu().numpy(), bias, k, True)
        gi, gs = B.moe_gate_topk(x, wg, to_dev(bias, torch.float32), k, True)
        torch.cuda.synchronize()
        assert np.array_equal(gi.cpu().numpy(), oi)
        assert np.allclose(gs.cpu().numpy(), osc, rtol=1e-5, atol=1e-9)
