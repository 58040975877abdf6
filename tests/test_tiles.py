"""Views whose tiles are not 64x64: wide tiles (one tile where 64x64 tiles would
take several), ragged ones and rows that are no whole number of 16-byte stores."""
import dataclasses
import functools

import numpy as np
import pytest

from oracle import oracle as O
from paper_2607_26005_amd import scenegen as sg
from tests.parity import assert_parity


def test_row_split_is_exact_for_every_tile():
    # the write-out's u / n = (u * ceil(2^16 / n)) >> 16, for every tile that fits
    # the 64 x 68-word framebuffer (rows of roundup8(w) + 4 words)
    for w in range(1, 129):
        for h in range(1, 129):
            if (-(-w // 8) * 8 + 4) * (-(-h // 8) * 8) > 64 * 68:
                continue
            for d in (4, 16):
                if w % d == 0:
                    n = w // d
                    u = np.arange(n * h)
                    assert np.array_equal((u * ((65535 + n) // n)) >> 16, u // n), (w, h, d)


def test_block_row_split_is_exact():
    # b / n = (b * (floor(65536 / n) + 1)) >> 16 for the block tests of a wide tile,
    # also when the reciprocal's error takes the quotient one lower
    b = np.arange(256)
    for n in range(1, 17):
        for r in (65536 // n + 1, int(65536 / n * (1 - 2e-7)) + 1):
            assert np.array_equal((b * r) >> 16, b // n), (n, r)


@functools.lru_cache(maxsize=None)
def workload(cfg, worlds):
    return sg.make_config(cfg, num_worlds=worlds)


SIZES = [(100, 75, 0.3), (80, 45, 0.0), (65, 65, 0.0), (96, 96, 0.0), (120, 67, 0.25), (128, 32, 0.0), (128, 33, 0.0),
         (68, 64, 0.0), (30, 120, 0.0), (52, 38, 0.0), (61, 7, 0.0), (4, 4, 0.0), (1, 1, 0.0), (130, 50, 0.0), (136, 76, 0.25)]


@pytest.mark.gpu
@pytest.mark.parametrize("w, h, shift", SIZES)
@pytest.mark.parametrize("mode", ["class", "colour", "antialiased", "instances"])
@pytest.mark.parametrize("worlds", [1, 12])   # tiles cut into columns; whole and (from 8,192 tiles on) wide ones
def test_tiles_match_the_oracle(mode, w, h, shift, worlds):
    import torch
    from paper_2607_26005_amd import pictura
    wl = workload(7 if h % 2 else 3, worlds)   # town with lights, or dense traffic
    if worlds > 1 and (w > 64 or h > 64) and w * h < 16000:   # eight cameras: a launch of wide tiles
        wl = dataclasses.replace(wl, rig=dataclasses.replace(wl.rig, mount=np.concatenate([wl.rig.mount] * 2)))
        if wl.num_views < 5000:   # (the town has fewer agents: each stands three times in its world)
            a = wl.agents
            thrice = lambda v: np.repeat(v.reshape(a.num_worlds, -1), 3, 0).reshape(-1)
            wl = dataclasses.replace(wl, agents=dataclasses.replace(
                a, agents_per_world=3 * a.agents_per_world, **{f.name: thrice(getattr(a, f.name)) for f in dataclasses.fields(a)
                                                               if isinstance(getattr(a, f.name), np.ndarray)}))
    rig = dataclasses.replace(wl.rig, width=w, height=h, fx=0.6 * w, fy=0.6 * w, cx=w / 2.0 + shift,
                              cy=h / 2.0 - shift)
    print(f"[{mode}] {w}x{h}", flush=True)
    r = pictura.Renderer(0)
    try:
        r.upload(wl.scene, wl.cell_size)
        if wl.lights is not None:
            r.set_lights(pictura.DeviceLights.from_host(wl.lights))
        da = pictura.DeviceAgents.from_host(wl.agents)
        V = wl.agents.count * rig.num_cams
        # the buffers end with a guard that the render must not touch
        n = V * h * w
        cls = torch.full((n + 4096,), 77, dtype=torch.uint8, device="cuda")
        depth = torch.full((n + 4096,), -7.0, dtype=torch.float32, device="cuda")
        views = np.sort(np.random.default_rng(w * 131 + h).choice(V, 12, replace=False))
        idx = torch.as_tensor(views, device="cuda")
        extra = {}
        if mode == "class":
            pictura.pictura_render_views(r.ctx, da, rig, cls, depth)
        elif mode == "instances":
            inst = torch.full((n + 4096,), 77, dtype=torch.int32, device="cuda")
            counts = torch.empty((V, wl.agents.agents_per_world, 2), dtype=torch.int32, device="cuda")
            pictura.pictura_render_instances(r.ctx, da, rig, cls, depth, inst, counts)
            assert (inst[n:] == 77).all()
            extra = {"inst": inst[:n].view(V, h, w)[idx].cpu().numpy(), "counts": counts[idx].cpu().numpy().view(np.uint32)}
        else:
            rgb = torch.full((3 * n + 4096,), 77, dtype=torch.uint8, device="cuda")
            fn = pictura.pictura_render_rgb if mode == "colour" else pictura.pictura_render_rgb_aa
            fn(r.ctx, da, rig, cls, depth, rgb)
            assert (rgb[3 * n:] == 77).all()
            extra = {"rgb": rgb[:3 * n].view(V, 3, h, w)[idx].cpu().numpy()}
        assert (cls[n:] == 77).all() and (depth[n:] == -7.0).all()
        got_c, got_d = (t[:n].view(V, h, w)[idx].cpu().numpy() for t in (cls, depth))
    finally:
        r.close_checked()
    ora = O.render(wl.scene, wl.agents, rig, view_ids=views, lights=wl.lights, want_instances=mode == "instances",
                   **({"want_rgb": True, "antialias": mode == "antialiased"} if mode in ("colour", "antialiased") else {}))
    assert_parity(got_c, got_d, ora, f"{mode} {w}x{h}")
    for k, v in extra.items():
        assert np.array_equal(v, ora[k]), (mode, w, h, k)


@pytest.mark.gpu
@pytest.mark.parametrize("mode, cfg, w, h, worlds, tiles", [
    ("class", 3, 96, 96, 12, 4), ("class", 3, 100, 100, 12, 4), ("class", 3, 150, 100, 12, 6),   # 3, 3 and 5 wide ones
    ("class", 3, 100, 75, 12, 2), ("class", 3, 100, 75, 3, 2), ("instances", 3, 100, 75, 3, 4),   # 12,288 and 3,072 views
    ("instances", 3, 100, 75, 4, 2), ("class", 3, 130, 50, 12, 2), ("antialiased", 3, 80, 45, 7, 1),
    ("antialiased", 7, 150, 100, 5, 5), ("class", 7, 96, 96, 16, 3)])   # lights
def test_wide_tiles_where_they_pay(mode, cfg, w, h, worlds, tiles):
    import torch
    from paper_2607_26005_amd import pictura
    wl = workload(cfg, worlds)
    mount = np.concatenate([wl.rig.mount] * 2)
    rig = dataclasses.replace(wl.rig, width=w, height=h, fx=0.6 * w, fy=0.6 * w, cx=w / 2.0, cy=h / 2.0, mount=mount)
    r = pictura.Renderer(0)
    try:
        r.upload(wl.scene, wl.cell_size)
        if wl.lights is not None:
            r.set_lights(pictura.DeviceLights.from_host(wl.lights))
        r.set_option(pictura.OPT_STATS, 1)
        da = pictura.DeviceAgents.from_host(wl.agents)
        if mode == "class":
            r.render(da, rig)
        elif mode == "instances":
            r.render_instances(da, rig)
        else:
            r.render_rgb(da, rig, antialias=True)
        assert pictura.pictura_stats_copy(r.ctx)["view_tiles"] == tiles * wl.agents.count * len(mount)
    finally:
        r.close_checked()
