"""Quantiser units at their edges: a unit shorter than, as long as and longer than the registers of the wavefronts that share it,
units that do not fill a workgroup, both widths, with channels of zeros, of subnormal scales (some units and one unit in the last
place), of a scale that rounds to zero and of infinite ones (from finite and from infinite weights).  Codes, scales and packed bytes
are compared bit for bit; the packed bytes are unpacked on the host from the layout's definition."""
import numpy as np
import pytest
import torch

import oracle
from helpers import to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


def _unpack(packed, E, K, N, bits):
    """Signed codes [E,K,N] from the fragment layout (moe_common.h)."""
    fk = 64 if bits == 4 else 32
    b = packed.reshape(E, N // 32, K // fk, 2, 32, 16)              # [expert][slab][block][half][channel][byte]
    if bits == 8:
        c = b.astype(np.int16).reshape(E, N // 32, K // fk, 2, 32, 2, 8) - 128         # byte 8 j + i
    else:
        nib = np.stack([b & 15, b >> 4], axis=-1).reshape(E, N // 32, K // fk, 2, 32, 4, 8).astype(np.int16) - 8
        c = nib[..., [0, 4, 1, 5, 2, 6, 3, 7]]                      # nibble position of index i
    # k = fk kb + 16 j + 8 half + i
    return c.transpose(0, 2, 5, 3, 6, 1, 4).reshape(E, K, N)


@pytest.mark.parametrize("bits,g,E,K,N", [
    (4, 64, 3, 64, 32), (8, 64, 1, 128, 96), (4, 128, 1, 384, 64), (8, 128, 3, 256, 32), (4, 192, 2, 384, 32), (8, 512, 1, 512, 64),
    (4, 0, 1, 640, 32), (8, 0, 2, 1024, 32), (4, 0, 1, 1088, 64), (8, 0, 1, 2048, 32), (4, 0, 1, 2112, 32), (8, 0, 1, 4160, 32)])
def test_quantize_units_bit_exact(bits, g, E, K, N):
    print(f"quantize units bits={bits} g={g} E={E} K={K} N={N}", flush=True)
    rng = np.random.default_rng(K + N + bits)
    w = (rng.standard_normal((E, K, N)) * 0.02).astype(np.float32)
    w[0, :, 3] = 0.0
    w[0, :, 4] *= np.float32(1e-3)                                  # subnormal scale
    w[0, :, 5] = rng.integers(-2 * 7, 2 * 7 + 1, K) * np.float32(0.5) * np.float32(2.0 ** -24)      # the smallest one, with ties
    w[0, 0::64, 5] = np.float32((2 ** (bits - 1) - 1) * 2.0 ** -24)
    w[0, :, 6] *= np.float32(1e-9)                                  # scale rounds to zero
    w[0, :, 9] *= np.float32(1e9)                                   # infinite scale: codes of zero
    w[0, 7, 10], w[0, K - 3, 10] = np.inf, -np.inf                  # ... from infinite weights, whose own code is the lowest
    w[E - 1, :, 8] = rng.integers(-2 * 7, 2 * 7 + 1, K) * np.float32(0.5) * np.float32(2.0 ** -6)      # ties
    w[E - 1, K // 2, 8] = np.float32((2 ** (bits - 1) - 1) * 2.0 ** -6)
    oq, os_ = oracle.quantize(w, bits, g)
    oq[np.isinf(w)] = -(2 ** (bits - 1) - 1)                        # (inf / inf, which the oracle's C leaves undefined)
    sc = os_.view(np.float16)[0]
    assert (sc[:, [4, 5]] > 0).all() and (sc[:, [4, 5]] < 2.0 ** -14).all() and (sc[:, 6] == 0).all() and np.isinf(sc[:, 9]).all() and np.isinf(sc[[0, -1], 10]).all()
    canon, scales, packed = B.moe_quantize_experts(to_dev(w, torch.float32), bits, g)
    none, scales2, packed2 = B.moe_quantize_experts(to_dev(w, torch.float32), bits, g, want_canon=False)
    only, _, no_packed = B.moe_quantize_experts(to_dev(w, torch.float32), bits, g, want_packed=False)
    torch.cuda.synchronize()
    want = oq if bits == 8 else oracle.pack_int4(oq)
    assert none is None and no_packed is None
    assert np.array_equal(canon.cpu().numpy().view(want.dtype), want) and torch.equal(canon, only)
    assert np.array_equal(scales.cpu().numpy().view(np.uint16), os_) and torch.equal(scales, scales2)
    assert torch.equal(packed, packed2)
    assert np.array_equal(_unpack(packed.cpu().numpy(), E, K, N, bits), oq)


# Units of more than 2048 rows of sixteen (more than 64 slabs) and of eight channels: rows that fill two or four blocks of a wavefront, and a last run of one, two
# or three of them; as many rows as the registers hold and more (read twice); a last group of eight slabs that is not full
@pytest.mark.parametrize("bits,g,E,K,N", [(4, 0, 1, 2112, 96), (8, 0, 1, 2176, 32), (4, 0, 1, 2304, 2112), (8, 0, 3, 2240, 704), (4, 0, 1, 8256, 64), (8, 0, 1, 8256, 32),
                                          (4, 4160, 1, 8320, 1056), (8, 2176, 2, 4352, 32)])
def test_parts_of_slabs_bit_exact(bits, g, E, K, N):
    test_quantize_units_bit_exact(bits, g, E, K, N)


@pytest.mark.parametrize("bits,g,E,K,N", [(4, 0, 17, 1024, 1024), (8, 128, 9, 768, 2560), (4, 0, 4, 2048, 2080), (8, 0, 2, 4096, 2112)])
def test_large_masters_give_the_bytes_of_their_experts(bits, g, E, K, N):
    """Masters of more than 64 MB are loaded non-temporal where the registers hold a unit: expert by expert they are not."""
    print(f"quantize large bits={bits} g={g} E={E} K={K} N={N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K + N)
    w = torch.randn((E, K, N), generator=gen, device="cuda") * 0.02
    canon, scales, packed = B.moe_quantize_experts(w, bits, g)
    packed2 = B.moe_quantize_experts(w, bits, g, want_canon=False)[2]
    for e in range(E):
        c, s, p = B.moe_quantize_experts(w[e:e + 1].contiguous(), bits, g)
        assert torch.equal(canon[e], c[0]) and torch.equal(scales[e], s[0]) and torch.equal(packed.view(E, -1)[e], p.view(-1))
    assert torch.equal(packed, packed2)
