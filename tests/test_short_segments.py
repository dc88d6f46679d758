"""Layouts of many short segments that stream: bit for bit the same buffers through handles that do not."""

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

import harness as H

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("rows,topology,params,grads,decay", [
    (4, "ring", "f32", "f32", True),           # cut tiles element by element: tile kernel
    (9, "exp", "f32", "bf16", False),          # by groups
    (17, "exp", "f32", "f32", True),
    (32, "complete", "f32", "f32", False),     # loop kernel, element by element
    (16, "complete", "f32", "f32", False),     # by groups
    (16, "complete", "bf16", "f32", True),
    (8, "ring", "bf16", "bf16", True),
    (40, "one_peer", "f32", "f32", True),      # accumulation by whole items, in order; mixing by the tile
    (90, "one_peer", "f32", "f32", False),
    (40, "one_peer", "bf16", "f32", False),    # accumulation by pieces
    (96, "exp", "f32", "f32", False),          # tile of sixteen wavefronts
    (96, "exp", "bf16", "bf16", True),         # steps direct, mixing by the tile
])
def test_short_segments_give_the_bits_of_small_handles(rows, topology, params, grads, decay):
    """Every phase of a step, a range, accumulation and mixing of segments of 1 to 2300 elements and one long one."""
    print("case", rows, topology, params, grads, decay, flush=True)
    dev = torch.device(DEV)
    chunk = (512 << 20) // (24 * rows) // 65536 * 65536          # the largest piece that does not stream
    sizes = [1 + 977 * k % 2300 for k in range((chunk + 70001) // 1160)] + [70001]
    layout = WL.pack([("t%d" % k, (n,)) for k, n in enumerate(sizes)])
    wd = [0.1 * (k % 2) for k in range(len(sizes))] if decay else None
    csr = {"ring": lambda: WL.ring(rows), "exp": lambda: WL.static_exponential(rows), "complete": lambda: WL.complete(rows),
           "one_peer": lambda: WL.one_peer_exponential(rows, 1)}[topology]()
    hp = H.HyperF32(s=2)
    sims = [H.GpuSim(rows, rows, layout, hp, [csr], params, grads, weight_decay=wd, pad_fill=777.0) for _ in range(2)]
    big, ref = sims
    assert B.dadam_get_plan_info(big.h).streaming == 1
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows)
    mask = torch.from_numpy(H.valid_mask(layout)).to(dev)
    noise = lambda std: torch.empty(layout.d, device=dev).normal_(0.0, std, generator=gen)
    for c in range(rows):
        # whole numbers over 16 or 32 rows of equal weights: the sums are exact, in whichever order a loop's wavefronts share them
        x = noise(0.5) if topology != "complete" else torch.randint(-8, 9, (layout.d,), device=dev, generator=gen).float()
        for sim in sims:
            sim.x_src[c].copy_(x)
            sim.x_src[c][~mask] = float("nan")
    grad = [noise(1e-2).to(H.TORCH_DT[grads]) for _ in range(rows)]
    for g in grad:
        g[~mask] = float("nan")
    xdt, gdt = [B.DADAM_BF16 if t == "bf16" else B.DADAM_F32 for t in (params, grads)]
    small = []
    ends = [int(o) + int(n) for o, n in zip(layout.offsets, layout.numels)]
    for lo in range(0, layout.d, chunk):
        hi = min(lo + chunk, layout.d)
        parts = [(max(int(o), lo), min(e, hi), 0.0 if wd is None else wd[k])
                 for k, (o, e) in enumerate(zip(layout.offsets, ends)) if int(o) < hi and e > lo]
        h = B.dadam_init(rows, rows, hi - lo, [a - lo for a, _, _ in parts], [b - a for a, b, _ in parts], xdt, gdt, hp.lr, hp.beta1,
                         hp.beta2, hp.eps, hp.s, device=0, weight_decay=[w for _, _, w in parts])
        assert B.dadam_get_plan_info(h).streaming == 0
        B.dadam_set_topology(h, 0, *csr)
        small.append((h, lo, hi))

    def on_small(call):
        for h, lo, hi in small:
            cut = lambda ts: [t[lo:hi] for t in ts]
            B.dadam_bind(h, cut(ref.x_src), cut(ref.x_dst), cut(ref.m), cut(ref.v), cut(ref.b))
            call(h, cut(grad))

    names = ("x_dst", "m", "v", "b")
    padding = {(name, i): getattr(big, name)[i][~mask].clone() for name in names for i in range(rows)}

    def same(what):
        torch.cuda.synchronize()
        for name in names:
            for i in range(rows):
                a, b = getattr(big, name)[i], getattr(ref, name)[i]
                assert torch.equal(a[mask], b[mask]), (what, name, i)
                assert torch.equal(a[~mask], padding[name, i]), (what, name, i)

    stream = B.current_stream()
    for t, flags in ((1, B.DADAM_FUSE_ACCUM), (2, B.DADAM_FUSE_ACCUM), (3, 0)):
        big.step(grad, t, 0, flags)
        on_small(lambda h, g: B.dadam_gossip_step(h, 0, g, t, flags, stream))
        same(("step", t))
    B.dadam_accumulate(big.h, grad, 3, stream)
    on_small(lambda h, g: B.dadam_accumulate(h, g, 3, stream))
    same("accumulate")
    big.mix(0, 0)
    on_small(lambda h, g: B.dadam_mix(h, 0, 0, stream))
    same("mix")
    B.dadam_gossip_step_range(big.h, 0, grad, 4, B.DADAM_FUSE_ACCUM, 0, len(sizes) // 2, stream)
    B.dadam_gossip_step_range(big.h, 0, grad, 4, B.DADAM_FUSE_ACCUM, len(sizes) // 2, len(sizes), stream)
    on_small(lambda h, g: B.dadam_gossip_step(h, 0, g, 4, B.DADAM_FUSE_ACCUM, stream))
    same("ranges")
    for h, _, _ in small:
        B.dadam_destroy(h)
    for sim in sims:
        sim.close()
