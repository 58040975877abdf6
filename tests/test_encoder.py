"""The image encoder on the CPU: what a user may do with the module."""
import io

import numpy as np
import torch

from paper_2607_26005_amd.encoder import ViewEncoder


def test_encoder_can_be_scripted():
    torch.manual_seed(4)
    enc = ViewEncoder(cams=2).eval()
    cls, depth = torch.randint(0, 14, (4, 20, 24), dtype=torch.uint8), torch.rand(4, 20, 24) + 0.5
    ref = enc(cls, depth)
    scripted = torch.jit.script(enc)
    assert torch.equal(scripted(cls, depth), ref)
    buf = io.BytesIO()
    torch.jit.save(scripted, buf)
    buf.seek(0)
    assert torch.equal(torch.jit.load(buf)(cls, depth), ref)


def test_three_part_products_leave_out_less_than_2_to_the_minus_22():
    # the kernels' cut of fp32 values into bf16 parts: weights by truncation,
    # activations to the nearest; of the nine part products the three smallest
    # are left out
    def bits(x):
        return x.astype(np.float32).view(np.uint32)

    def trunc(x):
        return (bits(x) & np.uint32(0xFFFF0000)).view(np.float32)

    def nearest(x):
        u = bits(x)
        return ((u + np.uint32(0x7FFF) + ((u >> 16) & np.uint32(1))) & np.uint32(0xFFFF0000)).view(np.float32)

    def parts(x, cut):
        h = cut(np.minimum(x, np.float32(float.fromhex('0x1.FEp127'))))
        m = cut(x - h)
        l = cut((x - h) - m)
        assert np.array_equal(h.astype(np.float64) + m + l, x.astype(np.float64))
        return [p.astype(np.float64) for p in (h, m, l)]
    top = np.arange(0x7F7E0000, 0x7F800000, 37).astype(np.uint32).view(np.float32)
    parts(top, nearest)   # up to the largest number
    parts(top, trunc)
    rng = np.random.default_rng(0)
    edge = np.asarray([0, 1, 0x7F, 0x80, 0xFF, 0x7F7F, 0x7F80, 0x7FFF, 0x8000, 0x8080, 0x80FF, 0xFF7F, 0xFFFF], np.uint32)
    mant = np.concatenate([(edge[:, None] | (np.uint32(k) << 16)).ravel() for k in (0, 1, 0x3F, 0x7E, 0x7F)])
    value = lambda m: (np.uint32(0x3F800000) | m).view(np.float32)
    a, w = (v.ravel() for v in np.meshgrid(value(mant), value(mant)))
    n = 1 << 20
    a = np.concatenate([a, value(rng.integers(0, 1 << 23, n).astype(np.uint32))])
    w = np.concatenate([w, value(rng.integers(0, 1 << 23, n).astype(np.uint32))])
    pa, pw = parts(a, nearest), parts(w, trunc)
    left = pa[1] * pw[2] + pa[2] * pw[1] + pa[2] * pw[2]
    rel = left / (a.astype(np.float64) * w)
    assert np.abs(rel).max() < 2.0 ** -22
    assert abs(rel[-n:].mean()) < 2.0 ** -30   # random mantissas: either sign alike
