"""The end of a grouped GEMM tile (scale, bias, activation, gate scale, store): rows at the edges of the 32-row
tiles, a last column block that is only partly there, every output type, in both kernels with row tiles."""
import numpy as np
import pytest
import torch

import oracle
from helpers import MAX_ABS_TOL, ORC_DT, REL_L2_TOL, TORCH_DT, error_metrics, to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,bits,g,activation", [("f16", 4, 0, "relu"), ("f16", 8, 64, "gelu"), ("bf16", 8, 0, "gelu"), ("bf16", 4, 64, "relu")])
@pytest.mark.parametrize("rows,d,F,fc2", [([1, 31, 32, 0, 33], 320, 192, "ring"),              # the ring's 32-row blocks
                                          ([63, 64, 2, 65, 33], 320, 192, "ring"),             # its 64-row blocks, last ones with one live half
                                          ([129, 127, 96, 97], 2368, 2176, "ring"),
                                          # so many tiles in fc2 that it runs register-fed ones, of 32, 64 and 128 rows (8-bit, and at most 256
                                          # rows per expert: 64); a last column block that is partly there
                                          ([1, 31, 32, 0, 33] * 9, 2752, 192, "tiles"), ([63, 64, 2, 65, 33] * 3, 3392, 192, "tiles"),
                                          ([129, 127, 96, 97], 6208, 2176, "tiles"), ([300, 257, 290], 4160, 2112, "tiles")])
def test_tile_end_matches_oracle_in_every_output_type(act, bits, g, activation, rows, d, F, fc2):
    print(f"tile end {act} bits={bits} g={g} {activation} rows={rows} d={d} F={F}", flush=True)
    rng = np.random.default_rng(sum(rows) + bits + g)
    E, R = len(rows), sum(rows)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    x = to_dev(rng.standard_normal((R, d)).astype(np.float32), TORCH_DT[act])
    w1 = (rng.standard_normal((E, d, F)) * 0.02).astype(np.float32)
    w2 = (rng.standard_normal((E, F, d)) * 0.02).astype(np.float32)
    b1, b2 = (to_dev((rng.standard_normal((E, n)) * 0.1).astype(np.float32), torch.float16) for n in (F, d))
    _, s1, p1 = B.moe_quantize_experts(to_dev(w1, torch.float32), bits, g, want_canon=False)
    _, s2, p2 = B.moe_quantize_experts(to_dev(w2, torch.float32), bits, g, want_canon=False)
    y = {}
    for dt in (torch.float32, torch.float16, torch.bfloat16):
        y[dt] = B.moe_grouped_ffn_wq(x, to_dev(off, torch.int32), E, d, F, bits, g, p1, s1, p2, s2, b1=b1, b2=b2, y_dtype=dt,
                                     activation=activation)
        torch.cuda.synchronize()
    assert B.load().moe_last_ffn_kernels().decode().split()[1] == ("grouped_gemm_ring_kernel" if fc2 == "ring" else "grouped_gemm_kernel")
    # the 16-bit outputs are the fp32 one, rounded to nearest even: bit for bit
    assert torch.equal(y[torch.float16], y[torch.float32].half()) and torch.equal(y[torch.bfloat16], y[torch.float32].bfloat16())
    q1, o1 = oracle.quantize(w1, bits, g)
    q2, o2 = oracle.quantize(w2, bits, g)
    want = oracle.grouped_ffn(x.float().cpu().numpy(), off, q1, o1, q2, o2, g, ORC_DT[act], b1=b1.float().cpu().numpy(),
                              b2=b2.float().cpu().numpy(), activation=oracle.GELU if activation == "gelu" else oracle.RELU)
    max_abs, rel = error_metrics(y[torch.float32].cpu().numpy(), want)
    assert max_abs <= MAX_ABS_TOL and rel <= REL_L2_TOL
