"""The gate's chains, a lane per expert or two: features short of, at and past whole blocks of 128 and of the four partial sums (some with
none), experts that leave lanes empty, every number of tokens per lane at its edges, and rows too long for the LDS: the oracle's experts and its scales to
expf's accuracy, and the scales of the matrix-core form bit for bit."""
import numpy as np
import pytest
import torch

import launches as L
import oracle
from helpers import TORCH_DT, to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E", [(1, 8, 4), (5, 128, 8), (1024, 136, 12), (7, 1160, 16), (3, 4224, 16),
                                   (1, 120, 20), (9, 520, 28), (512, 1152, 32), (513, 640, 24), (1023, 72, 32),
                                   (1, 72, 36), (256, 512, 64), (257, 904, 52), (512, 1032, 60), (513, 4104, 64), (1024, 264, 44),
                                   (1, 64, 68), (255, 1536, 128), (259, 776, 100), (515, 392, 124),
                                   (4, 4352, 64), (514, 10248, 64), (6, 20488, 8)])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_gate_chains_bit_exact(T, d, E, act):
    print(f"gate chains T={T} d={d} E={E} {act}", flush=True)
    (call,) = L.record([L.gate(T, d, E, B._DT[TORCH_DT[act]])])
    name = call.launches[0].kernel
    if d < 20000 and not (act == "bf16" and 16 < E <= 32 and T > 512):
        assert name.startswith("gate_lanes_kernel_wide<" if E > 64 else "gate_token_kernel<"), name
    rng = np.random.default_rng(T + d + E)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), TORCH_DT[act])
    wg = to_dev((rng.standard_normal((d, E)) * 0.05).astype(np.float32), TORCH_DT[act])
    bias = (rng.standard_normal(E) * 0.05).astype(np.float32)
    fin = (rng.random(T) < 0.2).astype(np.uint8)
    for k, renorm in ((1, True), (2, True), (2, False)):
        oi, osc = oracle.gate(x.float().cpu().numpy(), wg.float().cpu().numpy(), bias, k, renorm, finished=fin)
        gi, gs = B.moe_gate_topk(x, wg, to_dev(bias, torch.float32), k, renorm, finished=to_dev(fin, torch.uint8))
        torch.cuda.synchronize()
        assert np.array_equal(gi.cpu().numpy(), oi)
        assert np.allclose(gs.cpu().numpy(), osc, rtol=1e-5, atol=1e-9)         # (expf)


# ... bit for bit: the renormalised scales of two experts come from their two logits alone, and a batch too large for the chains takes the matrix cores, whose
# order of additions is the contract's.  Every number of experts per form at its edges, whole blocks of features, and short ones of one octet to fifteen.
@pytest.mark.parametrize("T,d,E", [(1, 512, 4), (1000, 8, 4), (77, 632, 8), (5, 1272, 12), (33, 2048, 16), (128, 248, 16), (3, 376, 20), (511, 504, 32), (600, 1016, 24),
                                   (2, 120, 36), (300, 888, 64), (700, 1032, 48), (900, 384, 40), (1, 128, 68), (256, 1016, 128), (19, 568, 100), (400, 264, 96),
                                   (520, 2048, 128), (513, 64, 124)])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_chains_give_the_bits_of_the_matrix_cores(T, d, E, act):
    print(f"gate chains, bits T={T} d={d} E={E} {act}", flush=True)
    n = -(-1100 // T)
    small, large = (c.launches[0].kernel for c in L.record([L.gate(t, d, E, B._DT[TORCH_DT[act]]) for t in (T, T * n)]))
    assert large.startswith("gate_mfma_kernel<")
    if not (act == "bf16" and T > 512 and 16 < E <= 64):
        assert small.startswith("gate_lanes_kernel_wide<" if E > 64 else "gate_token_kernel<"), small
    rng = np.random.default_rng(T + d + E)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), TORCH_DT[act])
    wg = to_dev((rng.standard_normal((d, E)) * 0.05).astype(np.float32), TORCH_DT[act])
    bias = to_dev((rng.standard_normal(E) * 0.05).astype(np.float32), torch.float32)
    si, ss = B.moe_gate_topk(x, wg, bias, 2, True)
    bi, bs = B.moe_gate_topk(x.repeat(n, 1), wg, bias, 2, True)
    torch.cuda.synchronize()
    assert torch.equal(si.repeat(n, 1), bi) and torch.equal(ss.repeat(n, 1), bs)
    # experts far apart: every logit of the first four decides a scale once
    for e in range(min(E, 4)):
        lift = bias.clone()
        lift[[e, E - 1 - e]] += 40.0
        if e != E - 1 - e:
            (ai, a), (ci, c) = B.moe_gate_topk(x, wg, lift, 2, True), B.moe_gate_topk(x.repeat(n, 1), wg, lift, 2, True)
            torch.cuda.synchronize()
            assert set(ai.unique().tolist()) == {e, E - 1 - e} and torch.equal(ai.repeat(n, 1), ci) and torch.equal(a.repeat(n, 1), c)
