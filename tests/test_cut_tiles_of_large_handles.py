"""Streaming launches of handles with their tables in device memory, which load cut tiles element by element and begin with the last one: bit for bit
against handles over parts of the same elements, which do not stream.  Padding is NaN on input and must keep a sentinel."""

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

import harness as H


@pytest.mark.gpu
@pytest.mark.parametrize("kind,rows,params,grads,decay", [("exp", 72, "f32", "f32", True), ("exp", 96, "bf16", "bf16", False), ("ring", 130, "bf16", "f32", True),
                                                          ("exp", 80, "f32", "bf16", False), ("exp", 66, "f32", "f32", False)])
@pytest.mark.parametrize("tail", [1, 6])
def test_streaming_cut_tiles(kind, rows, params, grads, decay, tail):
    print("case", kind, rows, params, grads, decay, tail, flush=True)
    dev = torch.device("cuda:0")
    # three tensors of some 120 thousand elements, cut inside a tile and, by tail, inside the last group of the buffer
    d = (512 << 20) // (24 * rows) // 4096 * 4096 + 4096
    sizes = [d // 3 // 8 * 8 - 3, d // 3 // 8 * 8 + 5]
    layout = WL.pack([("t%d" % k, (n,)) for k, n in enumerate(sizes + [d // 3 // 8 * 8 + tail])])
    offsets, numels = [int(o) for o in layout.offsets], [int(n) for n in layout.numels]
    d = offsets[-1] + numels[-1]                   # no padding behind the last tensor: its last group may be cut by the buffer's end
    wd = [0.1, 0.0, 0.05] if decay else None
    csr = {"exp": WL.static_exponential, "ring": WL.ring}[kind](rows)
    hp = H.HyperF32(s=2)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows)
    mask = torch.zeros(d, dtype=torch.bool, device=dev)
    for o, n in zip(offsets, numels):
        mask[o:o + n] = True

    def draw(dt, std, low=None):
        out = []
        for _ in range(rows):
            t = torch.empty(d, device=dev)
            t = t.normal_(0.0, std, generator=gen) if low is None else t.uniform_(low, std, generator=gen)
            t[~mask] = float("nan")
            out.append(t.to(dt))
        return out

    x, g = draw(H.TORCH_DT[params], 0.5), draw(H.TORCH_DT[grads], 1e-2)
    state = draw(torch.float32, 1e-3) + draw(torch.float32, 1e-4, 1e-5) + draw(torch.float32, 1e-3)
    results, errors = [], []
    for parts in ([(0, 3)], [(0, 1), (1, 2), (2, 3)]):
        out, mixed, now, error = [torch.full_like(t, 7.0) for t in x], [torch.full_like(t, 7.0) for t in x], [t.clone() for t in state], 0.0
        for first, last in parts:
            lo, hi = offsets[first], offsets[last - 1] + numels[last - 1]
            cut = lambda ts: [t[lo:hi] for t in ts]  # noqa: E731, B023
            h = B.dadam_init(rows, rows, hi - lo, [o - lo for o in offsets[first:last]], numels[first:last], H.ABI_DT[params], H.ABI_DT[grads], hp.lr,
                             hp.beta1, hp.beta2, hp.eps, hp.s, device=0, weight_decay=None if wd is None else wd[first:last])
            assert B.dadam_get_plan_info(h).streaming == (len(parts) == 1)
            B.dadam_set_topology(h, 0, *csr)
            B.dadam_bind(h, cut(x), cut(out), cut(now[:rows]), cut(now[rows:2 * rows]), cut(now[2 * rows:]))
            stream = B.current_stream()
            B.dadam_gossip_step(h, 0, cut(g), 4, B.DADAM_FUSE_ACCUM, stream)
            B.dadam_accumulate(h, cut(g), 6, stream)
            B.dadam_bind(h, cut(x), cut(mixed), cut(now[:rows]), cut(now[rows:2 * rows]), cut(now[2 * rows:]))
            e = torch.zeros(1, dtype=torch.float64, device=dev)
            B.dadam_mix_consensus(h, 0, e, 0, stream)
            torch.cuda.synchronize()
            error += float(e)
            B.dadam_destroy(h)
        results.append(out + mixed + now)
        errors.append(error)
    for k, (p, q) in enumerate(zip(*results)):
        assert torch.equal(p[mask], q[mask]), k
        assert bool((p[~mask] == 7.0).all() if k < 2 * rows else p[~mask].isnan().all()), k
    # partial sums of float32 squares over another division into tiles: a few roundings of 2^-24 in each of hundreds of sums
    assert np.isclose(errors[0], errors[1], rtol=1e-6) and errors[0] > 0
