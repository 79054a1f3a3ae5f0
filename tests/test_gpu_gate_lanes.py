"""The gate's forms for few tokens: a block per one, two or four tokens with 65 to 256 experts (all of a lane's experts in one load,
pairs, pairs of odd counts), the wide loads of 33 to 64, and the pairs of large batches."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TORCH_DT, to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E", [(1, 8, 66), (5, 136, 126), (256, 640, 128), (257, 1032, 128), (511, 520, 100), (512, 2048, 96), (513, 64, 128),
                                   (3, 200, 36), (7, 1032, 64), (1024, 72, 60),
                                   (5, 8, 33), (6, 136, 64), (256, 1032, 47), (257, 520, 47), (4, 136, 50),             # one expert per lane and around it
                                   (1, 8, 65), (5, 136, 127), (257, 640, 99), (1023, 264, 127), (1022, 128, 66),        # two experts per lane
                                   (1, 8, 129), (4, 1032, 255), (300, 520, 191), (1021, 72, 253),                       # four, odd counts
                                   (3, 200, 130), (256, 640, 254), (511, 136, 250), (2047, 64, 194),                    # ... in pairs
                                   (7, 1160, 132), (200, 512, 256), (513, 264, 200),                                    # ... in one load
                                   (2049, 72, 17), (2050, 200, 63), (2051, 64, 127), (2052, 136, 255),                  # matrix cores, odd counts
                                   (2053, 72, 62), (2054, 136, 126), (2055, 200, 250),                                  # ... pairs
                                   (8161, 72, 131), (8162, 136, 202)])                                                  # ... in two row tiles
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
