"""Layouts of many short tensors side by side, which run by one dense grid and a map of what is stored: on the CPU from the sources'
own text, and on the GPU bit for bit against a handle over the same tensors that has no map (one more tensor behind a wide gap)."""

import os
import re
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import build as bld
from paper_2410_11998_amd import workloads as WL
from test_host_abi import _route_answers

import harness as H


def test_a_map_has_what_the_segments_have(tmp_path):
    clang = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")
    if clang is None:
        pytest.skip("no clang++")
    src = open(os.path.join(bld.CSRC, "dadam_device.h")).read()
    b = src.index("// Algorithm 3, lines 6-13, for one element.")
    steps = src[src.index("template <bool STREAM>\nconstexpr int kGroupStep"):src.index("typedef float f4")]
    (tmp_path / "helpers.inc").write_text(steps + src[src.index("typedef float f4 __attribute__"):src.rindex("// ----", 0, b)])
    a = src.index("template <typename A>\n__device__ __forceinline__ int clip_of")
    (tmp_path / "clip.inc").write_text(src[a:src.index("// Pointers of the bound buffers.", a)])
    host = open(os.path.join(bld.CSRC, "dadam_host.cpp")).read()
    a = host.index("bool can_map(")
    (tmp_path / "host.inc").write_text(host[a:host.index("// Number the tiles of every tile grid.", a)])
    exe = str(tmp_path / "map")
    subprocess.run([clang, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I", str(tmp_path),
                    os.path.join(os.path.dirname(os.path.abspath(__file__)), "emulate_map.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout == ("bad 0, spread some, partial groups some\n"
                        "packed 1 one 0 gap7 1 gap8 0 d0 two decays 0 decay inside a group 0 long 0\n"), r.stdout


CASES = [
    (1, "share", 5, "f32", "f32", True),             # direct, in place, launches of a few pieces
    (1, "share", 5, "bf16", "f32", True),
    (8, "ring", 300, "bf16", "f32", True),           # tile kernel
    (5, "ring", 300, "f32", "bf16", False),
    (2, "ring", 8400, "f32", "f32", True),           # streams in steps alone, by the mixing tile's shape
    (16, "exp", 900, "bf16", "bf16", True),
    (20, "exp", 3, "f32", "f32", True),              # few tiles: row by row
    (32, "complete", 700, "f32", "f32", True),       # loops
    (32, "complete", 700, "bf16", "bf16", False),
    (70, "ring", 400, "bf16", "bf16", True),         # tables in device memory
    (96, "exp", 40, "f32", "f32", False),
    (24, "one_peer", 2900, "f32", "f32", True),      # streams: lanes spread inside the layout, two vectors
    (48, "one_peer", 1500, "f32", "f32", True),      # steps row by row, mixing by whole items
    (40, "one_peer", 1500, "bf16", "bf16", True),
    (64, "complete", 900, "f32", "f32", False),      # loops that stream
    (72, "exp", 900, "f32", "f32", True),
]


def layouts(sizes, decay):
    """What both handles of a case lay out: `sizes` short tensors, and the same with one more behind a wide gap."""
    shapes = [("t%d" % k, (1 + 977 * k % 2300 if k % 5 else 1 + k % 11,)) for k in range(sizes)]
    layout = WL.pack(shapes)
    wd = [0.1 * (k % 2) for k in range(sizes)] if decay else None
    more = WL.PackedLayout(layout.names + ["last"], np.append(layout.offsets, np.uint64(layout.d + 16)), np.append(layout.numels, np.uint64(8)),
                           layout.d + 24)
    return layout, wd, more


def test_which_launches_go_by_the_map(tmp_path):
    """The layouts that the GPU test compares: every launch of the one handle has the map, none of the other; and on both sides of the lines from which
    launches go by long segments all the same.  Kernels of whole items for steps and accumulation store into padding: none has a map."""
    asked, want = "", {}
    for n, (rows, topology, sizes, params, _, decay) in enumerate(CASES):
        layout, wd, more = layouts(sizes, decay)
        for name, lay, decays, walk in (("map", layout, wd, "map"), ("segments", more, None if wd is None else wd + [0.0], None)):
            tensors = " ".join(f"{o} {k} {w}" for o, k, w in zip(lay.offsets, lay.numels, decays or [0.0] * len(lay.names)))
            asked += f"{name}{n} {rows} {3 if topology == 'share' else rows} {int(params == 'bf16')} {lay.d} {len(lay.names)} {tensors}\n"
            want[f"{name}{n}"] = ", ".join([walk] * 3) if walk else None
    got = _route_answers(tmp_path, "map_of", asked)
    assert set(got) == set(want)
    for name, answer in got.items():
        assert answer == want[name] if want[name] else re.fullmatch(r"\d+ segments(, \d+ segments){2}", answer), (name, answer)

    got = _route_answers(tmp_path, "maps")
    m, s = "map", "segments"
    want = {  # step, mixing, mixing with the error, accumulation
        "share1 of 3 f32 1100+4 0e6": (m, m, m), "share1 of 3 bf16 1100+4 0e6": (m, m, m), "ring8 of 3 bf16 1100+4 2e6": (m, m, m, m),
        "ring8 of 3 f32 1100+8 2e6": (s, s, s, s), "ring8 of 3 f32 70000+4 2e6": (s, s, s, s),
        "ring40 of 2 f32 1100+4 120e6": (m, "map whole", m, m), "ring40 of 2 f32 1100+12 120e6": ("segments whole", s, s, "segments whole"),
        "ring48 of 2 bf16 1100+4 120e6": (m, "map whole", m, m), "ring100 of 2 f32 1100+4 120e6": (m, "map whole", m, m),
        "complete32 of 32 f32 16380+4 205e6": (m, m, m, m), "complete32 of 32 f32 16388+4 205e6": (s, s, m, m),
        "complete32 of 32 f32 16388+4 190e6": (m, m, m, m), "complete32 of 32 f32 20484+4 81e6": (s, s, m, m),
        "complete32 of 32 f32 20476+4 81e6": (m, m, m, m), "complete32 of 32 f32 20484+4 79e6": (m, m, m, m),
        "complete64 of 64 bf16 20484+4 81e6": (m, s, s, m), "halves64 of 0 f32 2564+4 205e6": (m, s, m, m), "halves64 of 0 f32 2556+4 205e6": (m, m, m, m),
        "complete96 of 96 f32 2052+4 205e6": (m, s, m, m),
        "complete96 of 96 f32 2044+4 205e6": (m, m, m, m), "complete96 of 96 f32 6148+4 205e6": (s, s, m, m),
        "complete128 of 128 f32 6148+4 205e6": (s, m, m, m), "complete96 of 96 bf16 8200+4 205e6": (m, s, m, m),
        "complete96 of 96 bf16 8184+4 205e6": (m, m, m, m), "ring18 of 3 bf16 20004+4 205e6": (m, m, m, m),
        "ring24 of 3 bf16 4100+4 205e6": (m, s, s, m), "ring24 of 3 bf16 4092+4 205e6": (m, m, m, m), "ring32 of 3 bf16 2564+4 205e6": (m, s, s, m),
        "ring32 of 3 bf16 2556+4 205e6": (m, m, m, m), "ring48 of 3 bf16 12292+4 101e6": (m, s, s, m), "ring48 of 3 bf16 12284+4 101e6": (m, m, m, m),
        "ring48 of 3 bf16 20004+4 79e6": (m, m, m, m), "ring72 of 3 bf16 20004+4 205e6": (m, m, m, m), "ring32 of 3 f32 20004+4 205e6": (m, m, m, m),
        "ring96 of 7 f32 5124+4 205e6": (s, m, m, m), "ring96 of 7 f32 5116+4 205e6": (m, m, m, m), "ring72 of 7 f32 5124+4 205e6": (m, m, m, m),
        "ring96 of 7 f32 5124+4 190e6": (m, m, m, m),
    }
    assert got == {k: ", ".join(v) for k, v in want.items()}


@pytest.mark.gpu
@pytest.mark.parametrize("rows,topology,sizes,params,grads,decay", CASES)
def test_mapped_layouts_give_the_bits_of_segments(rows, topology, sizes, params, grads, decay):
    """Every phase, update alone, accumulation, mixing, the consensus error and ranges; padding holds NaN (inputs) and a sentinel."""
    print("case", rows, topology, sizes, params, grads, decay, flush=True)
    dev = torch.device("cuda:0")
    share = topology == "share"
    cols = 3 if share else rows
    layout, wd, more = layouts(sizes, decay)
    csr = {"ring": lambda: WL.ring(rows), "exp": lambda: WL.static_exponential(rows), "complete": lambda: WL.complete(rows),
           "share": WL.node_share_ring, "one_peer": lambda: WL.one_peer_exponential(rows, 1)}[topology]()
    hp = H.HyperF32(s=2)
    sims = [H.GpuSim(rows, cols, more, hp, [csr], params, grads, weight_decay=None if wd is None else wd + [0.0], inplace=share, pad_fill=777.0)
            for _ in range(2)]
    here, ref = sims
    d = layout.d
    h = B.dadam_init(rows, cols, d, layout.offsets, layout.numels, H.ABI_DT[params], H.ABI_DT[grads], hp.lr, hp.beta1, hp.beta2, hp.eps, hp.s,
                     device=0, weight_decay=wd)
    B.dadam_set_topology(h, 0, *csr)
    cut = lambda ts: [t[:d] for t in ts]
    B.dadam_bind(h, cut(here.x_src), cut(here.x_dst), cut(here.m), cut(here.v), cut(here.b))
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows + sizes)
    mask = torch.from_numpy(H.valid_mask(more)).to(dev)
    noise = lambda std: torch.empty(more.d, device=dev).normal_(0.0, std, generator=gen)
    for c in range(cols):
        # whole numbers over equal weights of a power of two: the sums are exact, in whichever order a loop's wavefronts share them
        x = noise(0.5) if topology != "complete" else torch.randint(-8, 9, (more.d,), device=dev, generator=gen).float()
        for sim in sims:
            sim.x_src[c].copy_(x)
            sim.x_src[c][~mask] = float("nan")
    grad = [noise(1e-2).to(H.TORCH_DT[grads]) for _ in range(rows)]
    for g in grad:
        g[~mask] = float("nan")
    inside = mask[:d].clone()
    names = ("x_dst", "m", "v", "b")
    raw = lambda t: t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)
    before = {(name, i): getattr(here, name)[i][:d][~inside].clone() for name in names for i in range(rows)}

    def same(what):
        torch.cuda.synchronize()
        for name in names:
            for i in range(rows):
                a, b = getattr(here, name)[i][:d], getattr(ref, name)[i][:d]
                assert torch.equal(raw(a[inside]), raw(b[inside])), (what, name, i)
                assert torch.equal(raw(a[~inside]), raw(before[name, i])), (what, "padding", name, i)

    stream = B.current_stream()
    for t, flags in ((1, B.DADAM_FUSE_ACCUM), (2, B.DADAM_FUSE_ACCUM), (3, 0)):
        B.dadam_gossip_step(h, 0, cut(grad), t, flags, stream)
        ref.step(grad, t, 0, flags)
        same(("step", t))
    B.dadam_accumulate(h, cut(grad), 3, stream)
    ref.accumulate(grad, 3)
    same("accumulate")
    third = sizes // 3
    for tb, te in ((third, sizes), (0, third)):
        B.dadam_gossip_step_range(h, 0, cut(grad), 4, B.DADAM_FUSE_ACCUM, tb, te, stream)
        ref.step_range(grad, 4, tb, te)
    same("ranges")
    if not share:
        B.dadam_mix(h, 0, 0, stream)
        ref.mix(0, 0)
        same("mix")
        B.dadam_mix(h, 0, B.DADAM_FORCE_TILE, stream)
        ref.mix(0, B.DADAM_FORCE_TILE)
        same("mix by the tile")
        out = torch.zeros(2, dtype=torch.float64, device=dev)
        B.dadam_mix_consensus(h, 0, out[:1], 0, stream)
        same("consensus")
        x = torch.stack([s[:d][inside].double() for s in here.x_src])
        want = float((x - x.mean(0)).square().sum())
        # float32 sums of at most 96 sources an element, added in double: 1e-5 is far above their rounding, far below one stray element
        assert abs(float(out[0]) - want) <= 1e-5 * want, (float(out[0]), want)
    B.dadam_destroy(h)
    for sim in sims:
        sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows,topology,params,each,total", [
    (32, "complete", "f32", 20003, 205_000_000),     # loops
    (96, "complete", "f32", 6200, 205_000_000),      # loops, tables in device memory
    (96, "exp", "f32", 5201, 205_000_000),           # steps by the tile
    (32, "ring", "bf16", 2603, 205_000_000),         # mixing by the tile, with the error and without
    (48, "ring", "bf16", 12401, 101_000_000),
])
def test_long_segments_of_a_layout_with_a_map(rows, topology, params, each, total):
    """Launches that go by the segments of a handle that has a map, whole and by ranges, against a handle that has none; padding as above."""
    print("case", rows, topology, params, each, total, flush=True)
    dev = torch.device("cuda:0")
    dt = H.TORCH_DT[params]
    layout = WL.pack([("t%d" % k, (each - k % 3,)) for k in range(total // rows // (each + 8))])
    d, n = layout.d, len(layout.names)
    wd = [0.0] * n if topology == "complete" else [0.1 * (k % 2) for k in range(n)]     # (large steps of loops with decay go by the tile)
    csr = {"ring": WL.ring, "exp": WL.static_exponential, "complete": WL.complete}[topology](rows)
    hp = H.HyperF32(s=2)
    inside = torch.from_numpy(H.valid_mask(layout)).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows + each)

    def draw(t, std):
        made = []
        for _ in range(rows):
            made.append(torch.full((d + 24,), float("nan"), dtype=t, device=dev))
            made[-1][:d][inside] = torch.empty(d, device=dev).normal_(0.0, std, generator=gen).to(t)[inside]
            made[-1][d + 16:] = 0.5
        return made

    x, g = draw(dt, 0.5), draw(dt, 1e-2)
    start = [torch.empty(d + 24, device=dev).normal_(0.0, 1e-3, generator=gen) for _ in range(3)]
    results = []
    for mapped in (True, False):
        size = d if mapped else d + 24
        cut = lambda ts: [t[:size] for t in ts]  # noqa: B023, E731
        out = [torch.full_like(t, 777.0) for t in x]
        state = [s.abs().clone() for s in start for _ in range(rows)]
        error = torch.zeros(1, dtype=torch.float64, device=dev)
        h = B.dadam_init(rows, rows, size, list(layout.offsets) + ([] if mapped else [d + 16]), list(layout.numels) + ([] if mapped else [8]),
                         H.ABI_DT[params], H.ABI_DT[params], hp.lr, hp.beta1, hp.beta2, hp.eps, hp.s, device=0,
                         weight_decay=wd + ([] if mapped else [0.0]))
        B.dadam_set_topology(h, 0, *csr)
        B.dadam_bind(h, cut(x), cut(out), cut(state[:rows]), cut(state[rows:2 * rows]), cut(state[2 * rows:]))
        stream = B.current_stream()
        kept = []
        if params == "f32":
            B.dadam_gossip_step(h, 0, cut(g), 1, B.DADAM_FUSE_ACCUM, stream)
            for k in ((n // 100, n), (0, n // 100)):     # the larger range goes by segments too, the other by the map
                B.dadam_gossip_step_range(h, 0, cut(g), 2, B.DADAM_FUSE_ACCUM, k[0], k[1], stream)
            torch.cuda.synchronize()
            kept += [t[:d].clone() for t in out]
        if topology != "exp":
            B.dadam_mix(h, 0, 0, stream)
            torch.cuda.synchronize()
            kept += [t[:d].clone() for t in out]
        if topology == "ring":
            for t in out:
                t.fill_(777.0)
            B.dadam_mix_consensus(h, 0, error, 0, stream)
            torch.cuda.synchronize()
            kept += [t[:d].clone() for t in out]
        B.dadam_destroy(h)
        results.append(kept + [t[:d] for t in state])
        if topology == "ring":
            mean = sum(t[:d][inside].double() for t in x) / rows
            want = float(sum((t[:d][inside].double() - mean).square().sum() for t in x))
            got = float(error[0])                        # (the reference's last tensor is the same everywhere)
            # float32 sums of at most 48 sources an element, added in double
            assert abs(got - want) <= 1e-5 * want, (got, want)
    for p, q in zip(*results):
        assert torch.equal(p, q)
