"""The GELU between the two GEMMs against 64 bits: what a layer with an identity-like second matrix returns, over the range of v,
with its ends (both signs of zero, large values, infinities and NaN)."""
import numpy as np
import pytest
import torch
from scipy.special import ndtr

from helpers import to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


def _gelu_of(v):
    """v [n] fp32 -> the layer's gelu(v): W1 and W2 are zero, v is b1 (fp16), y = b2 + 0: so h is read back through an identity W2."""
    n = 64
    E = (len(v) + n - 1) // n
    b1 = np.zeros((E, n), dtype=np.float16)
    b1.reshape(-1)[:len(v)] = v
    w1, w2 = np.zeros((E, n, n), dtype=np.float32), np.tile(np.eye(n, dtype=np.float32), (E, 1, 1))
    _, s1, p1 = B.moe_quantize_experts(to_dev(w1, torch.float32), 8, 0, want_canon=False)
    _, s2, p2 = B.moe_quantize_experts(to_dev(w2, torch.float32), 8, 0, want_canon=False)
    x = torch.zeros((E, n), dtype=torch.float16, device="cuda:0")
    off = torch.arange(E + 1, dtype=torch.int32, device="cuda:0")
    y = B.moe_grouped_ffn_wq(x, off, E, n, n, 8, 0, p1, s1, p2, s2, b1=to_dev(b1, torch.float16), y_dtype=torch.float32, activation="gelu")
    torch.cuda.synchronize()
    scale = float(s2.float()[0, 0, 0]) * 127.0                     # (an fp16 scale: the identity's ones are 127 * s2)
    return y.cpu().numpy().reshape(-1)[:len(v)] / scale


def test_gelu_over_its_range():
    v = np.concatenate([np.linspace(-9, 9, 6000), 2.0 ** -np.arange(1, 15), -(2.0 ** -np.arange(1, 15)), [0.0, -0.0, 40.0, -40.0, 6e4, -6e4]])
    v = v.astype(np.float16).astype(np.float64)
    got, want = _gelu_of(v), v * ndtr(v)
    # h is rounded to fp16 (2^-11 of its size, 2^-25 where it is subnormal); the fp32 GELU itself is exact to 4e-7
    assert (np.abs(got - want) <= np.abs(want) * 2.0 ** -11 * 1.01 + 2.0 ** -25 + 4e-7).all()


def test_gelu_at_infinities_and_nan():
    got = _gelu_of(np.array([1.0, np.nan] + [0.0] * 62 + [2.0] * 64))
    assert np.isnan(got[:64]).any() and np.isfinite(got[64:]).all()
    got = _gelu_of(np.array([np.inf] + [0.0] * 63))
    assert not np.isfinite(got[0])
