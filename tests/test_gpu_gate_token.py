"""The gate's chains for few tokens by 24 to 64 experts, a multiple of eight (a lane per expert, the weight through LDS up to 32, straight into registers
beyond): short and odd feature counts, partly filled lanes, odd numbers of tokens, the largest batches of one token per lane.  The chosen experts are the
oracle's; the logits are, bit for bit, those of the matrix-core form, whose order of additions is the contract's."""
import numpy as np
import pytest
import torch

import launches as L
import oracle
from helpers import TORCH_DT, to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E", [(1, 8, 24), (2, 136, 32), (3, 520, 32), (511, 512, 24), (512, 1032, 32), (5, 4096, 32), (1, 504, 40), (7, 1160, 48), (256, 640, 56),
                                   (255, 2048, 64), (4, 1544, 64)])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_gate_token_kernel_bit_exact(T, d, E, act):
    print(f"gate T={T} d={d} E={E} {act}", flush=True)
    (call,) = L.record([L.gate(T, d, E, B._DT[TORCH_DT[act]])])
    assert call.launches[0].kernel.startswith("gate_token_kernel")
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
        assert np.allclose(gs.cpu().numpy(), osc, rtol=1e-5, atol=1e-9)
    # a batch too large for this form: renormalised scales of two experts come from their two logits alone
    n = -(-1100 // T)
    (call,) = L.record([L.gate(T * n, d, E, B._DT[TORCH_DT[act]])])
    assert call.launches[0].kernel.startswith("gate_mfma_kernel")
    bi, bs = B.moe_gate_topk(x.repeat(n, 1), wg, to_dev(bias, torch.float32), 2, True)
    si, ss = B.moe_gate_topk(x, wg, to_dev(bias, torch.float32), 2, True)
    torch.cuda.synchronize()
    assert torch.equal(si.repeat(n, 1), bi) and torch.equal(ss.repeat(n, 1), bs)
