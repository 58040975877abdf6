"""Render calls of one context on two streams.  Render kernels read the agents'
arrays in place, and a call on another stream than the previous one runs behind
that call's kernels (an event wait on the device): what the second stream does
afterwards to the first call's agents or outputs cannot reach that call."""
import time

import numpy as np
import pytest

from paper_2607_26005_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def _workload():
    from paper_2607_26005_amd import pictura
    wl = sg.make_config(2, num_worlds=4)    # small-batch worlds: 512 views per call
    other = wl.agents.copy()
    rng = np.random.default_rng(7)
    # a second agent set: every agent moved and turned, so every view differs
    other.x = (other.x + rng.uniform(-30.0, 30.0, other.x.shape)).astype(np.float32)
    other.y = (other.y + rng.uniform(-30.0, 30.0, other.y.shape)).astype(np.float32)
    h = rng.uniform(-np.pi, np.pi, other.x.shape)
    other.cos_h = np.cos(h).astype(np.float32)
    other.sin_h = np.sin(h).astype(np.float32)
    return wl, [pictura.DeviceAgents.from_host(wl.agents), pictura.DeviceAgents.from_host(other)]


def _busy(torch, stream, ms=100.0):
    """Keep `stream` busy for about `ms` milliseconds."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(stream):
        torch.cuda._sleep(100000)
        a.record()
        torch.cuda._sleep(1000000)
        b.record()
        b.synchronize()
        torch.cuda._sleep(int(1e6 * ms / max(a.elapsed_time(b), 1e-3)))


def test_render_calls_on_two_streams_keep_their_agents():
    torch = _torch()
    from paper_2607_26005_amd import pictura
    wl, sets = _workload()
    r = pictura.Renderer(0)
    try:
        r.upload(wl.scene, wl.cell_size)
        refs = [tuple(t.clone() for t in r.render(d, wl.rig)) for d in sets]
        torch.cuda.synchronize()
        assert not torch.equal(refs[0][0], refs[1][0])
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]   # default priority
        outs = []
        for rep in range(4):
            for i in (0, 1):
                outs.append((i, r.render(sets[i], wl.rig, stream=streams[i])))
        torch.cuda.synchronize()
        for i, (c, d) in outs:
            assert torch.equal(c, refs[i][0]), f"class image of agent set {i} changed on its stream"
            assert torch.equal(d, refs[i][1]), f"depth image of agent set {i} changed on its stream"
    finally:
        r.close_checked()


def test_instance_renders_on_two_streams_share_their_outputs():
    # the second call clears the counts of the same buffers: only behind the
    # first call's kernel, which adds to them
    torch = _torch()
    from paper_2607_26005_amd import pictura
    wl, sets = _workload()
    r = pictura.Renderer(0)
    try:
        r.upload(wl.scene, wl.cell_size)
        outs = r.render_instances(sets[0], wl.rig)
        first = [t.clone() for t in outs]
        refs = [t.clone() for t in r.render_instances(sets[1], wl.rig)]
        torch.cuda.synchronize()
        assert not torch.equal(first[3], refs[3])
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        _busy(torch, s1)   # the first call has not begun when the second is queued
        pictura.pictura_render_instances(r.ctx, sets[0], wl.rig, *outs, stream=s1)
        pictura.pictura_render_instances(r.ctx, sets[1], wl.rig, *outs, stream=s2)
        torch.cuda.synchronize()
        for got, want, name in zip(outs, refs, ("classes", "depths", "instances", "counts")):
            assert torch.equal(got, want), name
    finally:
        r.close_checked()


def test_render_on_another_stream_waits_for_the_last_one():
    # agents overwritten on the second stream, behind that stream's own render:
    # the render on the first stream, which reads them in place, has already ended
    torch = _torch()
    from paper_2607_26005_amd import pictura
    wl, sets = _workload()
    r = pictura.Renderer(0)
    try:
        r.upload(wl.scene, wl.cell_size)
        refs = [tuple(t.clone() for t in r.render(d, wl.rig)) for d in sets]
        torch.cuda.synchronize()
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        outs = [tuple(torch.empty_like(t) for t in refs[0]) for _ in sets]
        torch.cuda.synchronize()
        _busy(torch, s1)
        r.render(sets[0], wl.rig, *outs[0], stream=s1)
        r.render(sets[1], wl.rig, *outs[1], stream=s2)
        with torch.cuda.stream(s2):
            for f in ("x", "y", "cos_h", "sin_h"):
                getattr(sets[0], f).copy_(getattr(sets[1], f))
        torch.cuda.synchronize()
        for k in (0, 1):
            assert torch.equal(outs[k][0], refs[k][0]) and torch.equal(outs[k][1], refs[k][1]), k
    finally:
        r.close_checked()


def test_first_scene_of_a_context_waits_for_its_stream_only():
    torch = _torch()
    from paper_2607_26005_amd import pictura
    wl, sets = _workload()
    w = pictura.Renderer(0)   # kernels loaded, streams in use
    r = pictura.Renderer(0)
    try:
        w.upload(wl.scene, wl.cell_size)
        refs = w.render(sets[0], wl.rig)
        busy = torch.cuda.Stream()
        tiny = torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        _busy(torch, busy, 1000.0)
        for _ in range(8):   # a stream that does not share the busy one's hardware queue
            s = torch.cuda.Stream()
            e = torch.cuda.Event()
            with torch.cuda.stream(s):
                tiny.add_(1.0)
                e.record()
            for _ in range(100):
                if e.query():
                    break
                time.sleep(0.0002)
            if e.query():
                break
        assert not busy.query(), "a stream that runs beside the busy one"
        r.upload(wl.scene, wl.cell_size, stream=s)
        out = r.render(sets[0], wl.rig, stream=s)
        s.synchronize()
        assert not busy.query()
        torch.cuda.synchronize()
        assert torch.equal(out[0], refs[0]) and torch.equal(out[1], refs[1])
    finally:
        w.close_checked()
        r.close_checked()
