"""The image encoder on the CPU: what a user may do with the module."""
import io

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
