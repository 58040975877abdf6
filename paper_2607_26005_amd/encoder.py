"""Consumer of the rendered views: the perspective policy's image encoder, run on
the device straight from the renderer's output tensors, with no host round trip.

The paper couples its rasterizer with the policy inside one training process:
rendered views feed the network on the device (Sec. 3.2), where a small
from-scratch convolution stack encodes each camera view and learned query tokens
cross-attend over its feature map (Sec. 3.3, policy architecture; App. table of
architecture details: 4 cameras at 96x54, 5 convolution layers with 128 output
channels, 16 queries per camera and one cross-attention block, a 512-d scene
embedding).  The paper's views are RGB; here a view is what this renderer writes:
its class image (one channel per class) and its inverse depth (0 for sky).

The weights are random (the paper's trained weights are not available).  Inference
on the device runs in the library's kernels (csrc/pictura_encoder.hip); training
and every other use go through PyTorch's layers.
"""
from __future__ import annotations

import torch
import torch.nn as nn
import torch.nn.functional as F

NUM_CLASSES = 11   # ground .. light_green (scenegen.CLASS_NAMES)


class ViewEncoder(nn.Module):
    def __init__(self, cams: int = 4, width: int = 128, queries: int = 16, num_classes: int = NUM_CLASSES):
        super().__init__()
        self.cams, self.width, self.num_classes = cams, width, num_classes
        chans = [num_classes + 1, 32, 64, 64, 128, width]
        strides = [2, 2, 1, 2, 1]
        self.convs = nn.ModuleList(nn.Conv2d(chans[i], chans[i + 1], 3, stride=strides[i], padding=1)
                                   for i in range(5))
        self.queries = nn.Parameter(torch.randn(cams, queries, width) * 0.02)
        self.attn = nn.MultiheadAttention(width, 4, batch_first=True)
        self.proj = nn.Linear(width, width)

    def planes(self, cls: torch.Tensor, depth: torch.Tensor) -> torch.Tensor:
        """[V, H, W] uint8 classes and fp32 depths -> [V, classes + 1, H, W] inputs."""
        # (an elementwise comparison: F.one_hot would check the value range on the host)
        ids = torch.arange(self.num_classes, device=cls.device, dtype=torch.int32).view(1, -1, 1, 1)
        onehot = (cls.to(torch.int32).unsqueeze(1) == ids).to(torch.float32)
        inv = torch.reciprocal(depth).unsqueeze(1)   # +inf (sky) -> 0
        return torch.cat([onehot, inv], 1)

    @torch.jit.unused
    def _native(self, cls: torch.Tensor, depth: torch.Tensor) -> bool:
        """Whether the library's inference kernels compute this call: plain fp32
        weights of the shapes built above, rendered views on the device, nothing
        recorded or transformed on the way (gradients, autocast, tracing, functorch,
        dispatch modes, hooks)."""
        if type(cls) is not torch.Tensor or type(depth) is not torch.Tensor or type(self) is not ViewEncoder:
            return False
        if not (cls.is_cuda and cls.dtype == torch.uint8 and depth.dtype == torch.float32 and cls.dim() == 3
                and cls.shape == depth.shape and cls.device == depth.device and cls.is_contiguous()
                and depth.is_contiguous() and not depth.is_neg()):
            return False
        V, H, W = cls.shape
        if (V == 0 or V % self.cams or not (1 <= H <= 4096 and 1 <= W <= 4096) or not 1 <= self.cams <= 4096
                or not 1 <= self.num_classes <= 32):
            return False
        # One workgroup attends over a view's whole feature map, three times: few
        # large maps leave the chip idle, and from about 30,000 tokens the passes
        # come from memory.  Against the layers, views of 256x256 (1,024 tokens)
        # take 0.83 of the time for one and 0.94 for four, of 288x288 1.03 for two
        # and 1.05 for eight, of 512x512 1.16 for 8 and 0.77 for 24, of 1024x1024
        # (16,384) 1.03 for 16, 0.84 for 24 and 0.80 for 96, of 1920x1080 1.22-1.29
        # for 32-128, of 2048x2048 2.1.
        tokens = -(-H // 8) * -(-W // 8)
        if tokens > 1024 and (V < 24 or tokens > 16384):
            return False
        if (torch.compiler.is_compiling() or torch.jit.is_tracing() or torch.is_autocast_enabled("cuda")
                or torch._C._len_torch_dispatch_stack() or torch._C._len_torch_function_stack()
                or torch._C._functorch.peek_interpreter_stack() is not None
                or torch.autograd.forward_ad._current_level >= 0):
            return False
        mods = [self, *self.convs, self.attn, self.attn.out_proj, self.proj, self.convs]
        gm = nn.modules.module
        if gm._global_forward_hooks or gm._global_forward_pre_hooks or any(
                m._forward_hooks or m._forward_pre_hooks for m in mods[1:]) or any(
                "forward" in m.__dict__ for m in mods) or "planes" in self.__dict__:
            return False
        chans, strides = (self.num_classes + 1, 32, 64, 64, 128, 128), (2, 2, 1, 2, 1)
        a = self.attn
        if type(self.convs) is not nn.ModuleList or len(self.convs) != 5 or type(a) is not nn.MultiheadAttention \
                or type(self.proj) is not nn.Linear:
            return False
        for i, c in enumerate(self.convs):
            if (type(c) is not nn.Conv2d or c.weight.shape != (chans[i + 1], chans[i], 3, 3) or c.bias is None
                    or c.stride != (strides[i],) * 2 or c.padding != (1, 1) or c.dilation != (1, 1) or c.groups != 1
                    or c.padding_mode != "zeros"):
                return False
        if (a.num_heads != 4 or a.embed_dim != 128 or not a.batch_first or not a._qkv_same_embed_dim
                or a.in_proj_bias is None or a.out_proj.bias is None or a.bias_k is not None or a.add_zero_attn
                or (a.dropout and a.training) or self.queries.shape != (self.cams, 16, 128)
                or self.proj.weight.shape != (128, 128) or self.proj.bias is None):
            return False
        params = [self.queries, a.in_proj_weight, a.in_proj_bias, a.out_proj.weight, a.out_proj.bias, self.proj.weight,
                  self.proj.bias, *(p for c in self.convs for p in (c.weight, c.bias))]
        if any(type(p) not in (nn.Parameter, torch.Tensor) or p.dtype != torch.float32 or p.device != cls.device
               or not p.is_contiguous() or p.data_ptr() % 16 or p.is_neg() for p in params):
            return False
        return not torch.is_grad_enabled() or not (depth.requires_grad or any(p.requires_grad for p in params))

    @torch.jit.unused
    def _encode_native(self, cls: torch.Tensor, depth: torch.Tensor) -> torch.Tensor:
        from paper_2607_26005_amd import pictura
        a = self.attn
        with torch.cuda.device(cls.device):
            out = torch.empty((cls.shape[0], self.width), dtype=torch.float32, device=cls.device)
            pictura.pictura_encode_views(self.cams, self.num_classes, [(c.weight, c.bias) for c in self.convs],
                                         self.queries, (a.in_proj_weight, a.in_proj_bias),
                                         (a.out_proj.weight, a.out_proj.bias), (self.proj.weight, self.proj.bias),
                                         cls, depth, out)
        return out.reshape(cls.shape[0] // self.cams, self.cams * self.width)

    def forward(self, cls: torch.Tensor, depth: torch.Tensor) -> torch.Tensor:
        """cls, depth: [egos * cams, H, W], view v = ego * cams + camera.  Returns the
        [egos, cams * width] scene embedding (mean of each camera's pooled tokens)."""
        if not torch.jit.is_scripting():   # (a scripted module holds the layers alone)
            if self._native(cls, depth):
                return self._encode_native(cls, depth)
        x = self.planes(cls, depth)
        for conv in self.convs:
            x = F.relu(conv(x))
        V = x.shape[0]
        tokens = x.flatten(2).transpose(1, 2).contiguous()            # [V, h*w, width]
        q = self.queries.repeat(V // self.cams, 1, 1)                 # camera k's queries for view v
        pooled, _ = self.attn(q, tokens, tokens, need_weights=False)  # [V, queries, width]
        emb = self.proj(pooled.mean(1))                               # [V, width]
        return emb.reshape(V // self.cams, self.cams * self.width)
