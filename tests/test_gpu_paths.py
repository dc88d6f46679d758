"""Which kernel a launch takes, and what it computes, at the sizes where the choice changes: against the CPU
oracle, and where two kernels do the same sums in the same order, against each other bit for bit."""

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

import harness as H

pytestmark = pytest.mark.gpu


def rows_of_degree(n, deg):
    """n rows of `deg` sources each, spread over all n, weights summing to 1 in float32."""
    w = np.float32(1.0) / np.float32(deg)
    col = [(i + k * (k + 1) // 2) % n if deg <= 7 else (i + k) % n for i in range(n) for k in range(deg)]
    return np.arange(0, n * deg + 1, deg, dtype=np.int32), np.array(col, np.int32), np.full(n * deg, w, np.float32)


@pytest.mark.parametrize("n,deg,tiles,dtype", [
    (9, 3, 256, "f32"), (9, 3, 257, "f32"), (64, 7, 3, "f32"), (16, 6, 11, "bf16"), (12, 8, 5, "f32"),
    (13, 9, 2, "bf16"), (20, 12, 2, "f32"), (24, 15, 3, "f32"), (96, 68, 1, "f32"), (160, 71, 1, "bf16"),
])
def test_launches_of_few_tiles_give_the_tile_kernels_bits(n, deg, tiles, dtype):
    """Up to 256 tiles, more than eight rows run one wavefront per row and piece; the sums are those of the tile
    kernel, in the same order, for every length of the neighbour list (batches of eight, then four, then the rest,
    and a second chunk of the list beyond 64 entries)."""
    print("case", n, deg, tiles, dtype, flush=True)
    elems = 64 * (8 if dtype == "bf16" else 4)
    layout = WL.pack([("a", ((tiles - 1) * elems + 37,)), ("b", (elems - 60,))] if tiles > 1 else [("a", (elems - 3,))])
    csr = rows_of_degree(n, deg)
    hp = H.HyperF32(s=2)
    worst = H.run_parity(f"few-{n}-{deg}-{tiles}-{dtype}", n, n, layout, hp, [csr], lambda t: 0, 3, seed=77, param_dtype=dtype,
                         grad_dtype=dtype, flags=B.DADAM_FUSE_ACCUM, pad_fill=None)
    print("worst error / tolerance:", worst, flush=True)
    sims = [H.GpuSim(n, n, layout, hp, [csr], dtype, dtype) for _ in range(2)]
    for c in range(n):
        x0 = H.to_device(WL.normal_np(500 + c, layout.d, 0.02), dtype, "cuda:0")
        for sim in sims:
            sim.x_src[c].copy_(x0)
    for t in range(1, 4):
        grads = [H.to_device(WL.normal_np(600 + t * 200 + i, layout.d, 1e-3), dtype, "cuda:0") for i in range(n)]
        for sim, mode in zip(sims, (0, B.DADAM_FORCE_TILE)):
            sim.step(grads, t, 0, B.DADAM_FUSE_ACCUM | mode)
        torch.cuda.synchronize()
        for i in range(n):
            assert torch.equal(sims[0].x_dst[i], sims[1].x_dst[i]), (t, i)
            assert torch.equal(sims[0].m[i], sims[1].m[i]) and torch.equal(sims[0].b[i], sims[1].b[i])
        for sim in sims:
            sim.swap()
    for sim in sims:
        sim.close()


@pytest.mark.parametrize("deg,self_at,dtype", [(3, 2, "f32"), (2, None, "f32"), (9, 8, "bf16"), (9, None, "f32"), (14, 13, "f32")])
def test_weight_decay_finds_the_rows_own_parameters_wherever_the_list_has_them(deg, self_at, dtype):
    """The direct kernel keeps the row's own previous parameters from the mixing sum when the row lists itself, in
    any batch of the list, and loads them when it does not."""
    print("case", deg, self_at, dtype, flush=True)
    n = 16
    col = []
    for i in range(n):
        others = [(i + 1 + k) % n for k in range(deg)]
        if self_at is not None:
            others = others[:self_at] + [i] + others[self_at:deg - 1]
        col += others
    csr = (np.arange(0, n * deg + 1, deg, dtype=np.int32), np.array(col, np.int32), np.full(n * deg, np.float32(1) / np.float32(deg), np.float32))
    layout = WL.pack([("a", (530,)), ("b", (77,)), ("c", (1200,))])
    worst = H.run_parity(f"own-{deg}-{self_at}-{dtype}", n, n, layout, H.HyperF32(s=2), [csr], lambda t: 0, 3, seed=91, param_dtype=dtype,
                         grad_dtype=dtype, flags=B.DADAM_FUSE_ACCUM | B.DADAM_FORCE_DIRECT, weight_decay=[0.1, 0.0, 0.05])
    print("worst error / tolerance:", worst, flush=True)


@pytest.mark.parametrize("case", ["complete9", "complete8-bf16", "complete64", "complete33-decay", "aer32-inplace", "aer96", "aer24-bf16-decay",
                                  "gather-12x20", "broadcast-9", "weights-12", "complete160-bf16", "complete24-little-lds"])
def test_rows_of_a_loop_share_one_neighbour_sum(case):
    """The loop kernel against the oracle: loops of fewer and of more sources than a workgroup has wavefronts, several
    loops of different length, rows that all copy one source, unequal weights, sources that are no row's own, in place,
    with decay, on a ragged layout, in a whole accumulation loop."""
    print("case", case, flush=True)
    layout = WL.pack([("a", (1501,)), ("b", (5,)), ("c", (770,))])
    dtype = "bf16" if "bf16" in case else "f32"
    inplace, rng = "inplace" in case, np.random.default_rng(5)
    slot_of_t = lambda t: 0
    wd = [0.1, 0.0, 0.02] if "decay" in case else None
    if case.startswith("complete"):
        R = C = int(case[8:].split("-")[0])
        csrs = [WL.complete(R)]
    elif case.startswith("aer"):
        R = C = int(case[3:].split("-")[0])
        csrs, slot_of_t = [WL.aer(R // 4, k) for k in range(4)], lambda t: t % 4
    elif case.startswith("gather"):
        R, C = 12, 20
        csrs = [(np.arange(0, 37, 3, dtype=np.int32), np.tile(np.array([2, 19, 14], np.int32), 12), np.tile(np.array([0.5, 0.25, 0.25], np.float32), 12))]
    elif case.startswith("broadcast"):
        R = C = 9
        csrs = [(np.arange(10, dtype=np.int32), np.full(9, 4, np.int32), np.ones(9, np.float32))]
    else:                                # two loops of six rows with random weights, listed in a different order by every row
        R = C = 12
        w = (rng.random(6) + 0.1).astype(np.float32)
        w = (w / w.sum(dtype=np.float32)).astype(np.float32)
        col, ws = [], []
        for i in range(12):
            p = rng.permutation(6)
            col += [int(q) * 2 + i % 2 for q in p]
            ws += [w[q] for q in p]
        csrs = [(np.arange(0, 73, 6, dtype=np.int32), np.array(col, np.int32), np.array(ws, np.float32))]
    worst = H.run_parity(f"loop-{case}", R, C, layout, H.HyperF32(s=2), csrs, slot_of_t, 3, seed=88, param_dtype=dtype, grad_dtype=dtype,
                         flags=B.DADAM_FUSE_ACCUM, inplace=inplace, refresh_extra_sources=R != C, weight_decay=wd,
                         lds_limit_bytes=4096 if "little-lds" in case else 0,     # too little even for the partial sums: direct
                         pad_fill=None if inplace or C != R else 777.0, free_running=C == R)
    print("worst error / tolerance:", worst, flush=True)


@pytest.mark.parametrize("tiles", [512, 1030])            # 16 and 8 wavefronts
@pytest.mark.parametrize("sources", [1, 2, 3, 5, 6, 8, 9, 11, 13, 17, 20, 23, 24, 47, 48, 96])
def test_a_loops_shared_sum_is_as_accurate_as_the_listed_order(sources, tiles):
    """The order in which the loop kernel adds a loop's sources is no further from 64 bits than the tile kernel's chain
    of fused multiply-adds, whatever the number of sources; up to five are that chain."""
    print("case", sources, tiles, flush=True)
    R, d = 16, tiles * 256
    rng = np.random.default_rng(sources)
    w = (rng.random(sources) + 0.1).astype(np.float32)
    w = (w / w.sum(dtype=np.float64)).astype(np.float32)
    csr = (np.arange(0, R * sources + 1, sources, dtype=np.int32), np.tile(np.arange(sources, dtype=np.int32), R), np.tile(w, R))
    sim = H.GpuSim(R, sources, WL.pack([("a", (d,))]), H.HyperF32(s=1), [csr])
    for c in range(sources):
        sim.x_src[c].copy_(H.to_device(WL.normal_np(300 + c, d, 1.0), "f32", "cuda:0"))
    want = sum(float(w[c]) * sim.x_src[c].double() for c in range(sources))
    errors = []
    for flags in (0, B.DADAM_FORCE_TILE):
        sim.mix(0, flags)
        torch.cuda.synchronize()
        got = [x.clone() for x in sim.x_dst]
        assert all(torch.equal(x, got[0]) for x in got)
        errors.append((got[0], float((got[0].double() - want).square().mean().sqrt())))
    print("error of the shared sum / of the chain", errors[0][1], errors[1][1], flush=True)
    if sources <= 5:
        assert torch.equal(errors[0][0], errors[1][0])
    # 131072 elements: the ratio of the two means is known to better than 1 %
    assert errors[0][1] <= 1.01 * errors[1][1]
    sim.close()


@pytest.mark.parametrize("segments,rows,mode", [(2, 2, "tile"), (64, 2, "direct"), (65, 9, "auto"), (200, 4, "tile"), (4097, 2, "direct"),
                                                (4097, 64, "tile")])
def test_every_work_item_finds_its_segment(segments, rows, mode):
    """Layouts of many segments (contiguous tensors of a few elements whose weight decay alternates): the search by
    all lanes, 64 segments to a step, in small launches, and the binary search of large ones (64 rows)."""
    print("case", segments, rows, mode, flush=True)
    flag = {"tile": B.DADAM_FORCE_TILE, "direct": B.DADAM_FORCE_DIRECT, "auto": 0}[mode]
    layout = WL.pack([(f"t{k}", (1 + (7 * k) % 23,)) for k in range(segments)], align_elems=1)
    worst = H.run_parity(f"segments-{segments}-{rows}-{mode}", rows, rows, layout, H.HyperF32(s=2), [WL.ring(rows)], lambda t: 0, 2, seed=63,
                         flags=B.DADAM_FUSE_ACCUM | flag, weight_decay=[0.1 * (k % 2) for k in range(segments)], pad_fill=None)
    print("worst error / tolerance:", worst, flush=True)


def test_consensus_passes_follow_each_other_on_one_handle():
    """A pass leaves the handle's partial sums cleared for the next: repeated passes, also right behind a recorded one
    that has not run yet, report the same error as a fresh handle and as the entry point with the static array."""
    n, layout = 8, WL.pack([("a", (5003,)), ("b", (77,))])
    dev = torch.device("cuda:0")
    outs = torch.zeros(6, dtype=torch.float64, device=dev)
    sim = H.GpuSim(n, n, layout, H.HyperF32(s=2), [WL.ring(n)])
    for c in range(n):
        sim.x_src[c].copy_(H.to_device(WL.normal_np(900 + c, layout.d, 0.5), "f32", dev))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sim.mix_consensus(outs[0:1])
    for k in (1, 2):
        sim.mix_consensus(outs[k:k + 1])
    B.dadam_mix_consensus_static(sim.h, 0, outs[3:4], 0, sim.stream())
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
    sim.mix_consensus(outs[4:5])
    torch.cuda.synchronize()
    mask = H.valid_mask(layout)
    xs = [x.to(torch.float64).cpu().numpy()[mask] for x in sim.x_src]
    mean = sum(xs) / n
    want = sum(float(((x - mean) ** 2).sum()) for x in xs)
    got = [float(v) for v in outs[:5]]
    print("consensus errors", got, want, flush=True)
    assert all(abs(v - want) <= 1e-5 * want for v in got), (got, want)   # float32 per element (2^-24 x a few), double sums
    sim.close()


@pytest.mark.parametrize("rows,deg,dtype", [(24, 2, "f32"), (100, 3, "bf16"), (90, 8, "f32"), (96, 5, "bf16"), (20, 1, "f32")])
def test_large_mixing_of_rows_that_share_sources(rows, deg, dtype):
    """Mixing only, more than 1024 tiles and rows that stream directly: whole items by workgroups of four wavefronts,
    ragged ends included, against the tile kernel where it fits and against the sums in 64 bits."""
    print("case", rows, deg, dtype, flush=True)
    elems = 64 * (8 if dtype == "bf16" else 4)
    layout = WL.pack([("a", (1030 * elems + 13,)), ("b", (3 * elems - 5,)), ("c", (8 * elems,))])
    csr = rows_of_degree(rows, deg)
    if deg == 1:
        csr = (csr[0], np.array([i // 2 for i in range(rows)], np.int32), csr[2])   # two rows copy one source
    sim = H.GpuSim(rows, rows, layout, H.HyperF32(s=1), [csr], dtype, dtype)
    assert not B.dadam_slot_uses_tile_mode(sim.h, 0)
    for c in range(rows):
        sim.x_src[c].copy_(H.to_device(WL.normal_np(40 + c, layout.d, 0.5), dtype, "cuda:0"))
    for t in sim.x_dst:
        t.fill_(7.0)
    sim.mix(0, 0)
    torch.cuda.synchronize()
    mask = torch.from_numpy(H.valid_mask(layout)).to("cuda:0")
    for i in range(rows):
        want = torch.zeros(layout.d, dtype=torch.float64, device="cuda:0")
        size = torch.zeros_like(want)
        for k in range(csr[0][i], csr[0][i + 1]):
            x = sim.x_src[int(csr[1][k])].double()
            want += float(csr[2][k]) * x
            size += abs(float(csr[2][k])) * x.abs()
        err = (sim.x_dst[i].double() - want).abs()
        assert bool((err <= (1e-6 if dtype == "f32" else 1e-2) * size)[mask].all()), i     # a float32 sum; one bfloat16 rounding
        assert bool((sim.x_dst[i][~mask] == 7.0).all()), i
    got = [t.clone() for t in sim.x_dst]
    sim.mix(0, B.DADAM_FORCE_TILE)
    torch.cuda.synchronize()
    for i in range(rows):
        assert torch.equal(got[i], sim.x_dst[i]), i
    sim.close()


@pytest.mark.parametrize("rows,grads,s", [(33, "f32", 2), (40, "bf16", 3), (63, "f32", 1)])
def test_large_steps_by_whole_items_give_the_tile_kernels_bits(rows, grads, s):
    """Steps of 33 to 63 float32 rows in pairs over 1e8 elements go by whole items of four wavefronts, two vectors a lane:
    every phase, an update-only pass, decay, ragged ends and rows that do not divide among the dies, against the tile
    kernel, which does the same sums in the same order."""
    print("case", rows, grads, s, flush=True)
    d = 100_000_000 // rows + 2000
    layout = WL.pack([("a", (d - 1001,)), ("b", (5,)), ("c", (990,))])
    csr = rows_of_degree(rows, 2)
    sims = [H.GpuSim(rows, rows, layout, H.HyperF32(s=s), [csr], "f32", grads, weight_decay=[0.1, 0.0, 0.05], pad_fill=777.0) for _ in range(2)]
    assert not B.dadam_slot_uses_tile_mode(sims[0].h, 0)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    for c in range(rows):
        sims[0].x_src[c].normal_(0.0, 0.02, generator=gen)
        sims[1].x_src[c].copy_(sims[0].x_src[c])
    pool = [[torch.empty(layout.d, device=dev).normal_(0.0, 1e-2, generator=gen).to(H.TORCH_DT[grads]) for _ in range(rows)] for _ in range(2)]
    for t in range(1, 2 * s + 2):
        flags = B.DADAM_FUSE_ACCUM if t <= 2 * s else 0
        for sim, mode in zip(sims, (0, B.DADAM_FORCE_TILE)):
            sim.step(pool[t % 2], t, 0, flags | mode)
        torch.cuda.synchronize()
        for i in range(rows):
            for name in ("x_dst", "m", "v") + (("b",) if s > 1 else ()):
                assert torch.equal(getattr(sims[0], name)[i], getattr(sims[1], name)[i]), (t, i, name)
        for sim in sims:
            sim.swap()
    for sim in sims:
        sim.close()


@pytest.mark.parametrize("rows,params,grads,s", [(33, "f32", "f32", 3), (40, "bf16", "bf16", 2), (90, "bf16", "f32", 1), (127, "f32", "bf16", 2)])
def test_large_accumulation_by_whole_items(rows, params, grads, s):
    """Accumulation of 33 to 64 and 81 to 127 rows over 1e8 elements goes by whole items of four wavefronts: against the same call on
    a handle of the first row alone (one-wavefront pieces; elements never interact), bit for bit, ragged ends included."""
    print("case", rows, params, grads, s, flush=True)
    d = 100_000_000 // rows + 5000
    layout = WL.pack([("a", (d - 1001,)), ("b", (5,)), ("c", (990,))])
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    sim = H.GpuSim(rows, rows, layout, H.HyperF32(s=s), [WL.identity(rows)], params, grads, pad_fill=777.0)
    picked = (0, rows // 2, rows - 1)
    alone = [H.GpuSim(1, 1, layout, H.HyperF32(s=s), [WL.identity(1)], params, grads, pad_fill=777.0) for _ in picked]
    pool = [[torch.empty(layout.d, device=dev).normal_(0.0, 1e-2, generator=gen).to(H.TORCH_DT[grads]) for _ in range(rows)] for _ in range(2)]
    for t in range(1, 2 * s + 2):
        B.dadam_accumulate(sim.h, pool[t % 2], t, sim.stream())
        for one, i in zip(alone, picked):
            B.dadam_accumulate(one.h, [pool[t % 2][i]], t, one.stream())
        torch.cuda.synchronize()
        for one, i in zip(alone, picked):
            assert torch.equal(sim.m[i], one.m[0]) and torch.equal(sim.v[i], one.v[0]), (t, i)
            assert s == 1 or torch.equal(sim.b[i], one.b[0]), (t, i)
    # and the other rows against the recurrence itself in float64: b and m are sums of a few terms
    b, m = torch.zeros(layout.d, dtype=torch.float64, device=dev), torch.zeros(layout.d, dtype=torch.float64, device=dev)
    i, beta1 = 1, float(np.float32(0.9))
    for t in range(1, 2 * s + 2):
        b += pool[t % 2][i].double() / s
        if t % s == 0:
            m = beta1 * m + (1 - beta1) * b
            b.zero_()
    mask = torch.from_numpy(H.valid_mask(layout)).to(dev)
    assert float((sim.m[i].double() - m)[mask].abs().max()) < 1e-6 * 0.1       # |terms| below 0.1
    sim.close()
    for one in alone:
        one.close()


def rows_of_matrix(csr, i):
    return [(int(csr[1][k]), float(csr[2][k])) for k in range(csr[0][i], csr[0][i + 1])]


@pytest.mark.parametrize("kind,rows,tiles,params,grads,decay", [
    ("complete", 28, 520, "f32", "f32", False),            # 8 wavefronts, ordinary accesses
    ("complete", 60, 530, "f32", "f32", True),
    ("aer", 72, 200, "bf16", "f32", True),                 # the same with tables in device memory
    ("complete", 32, 2800, "f32", "f32", False),           # streaming
    ("aer", 64, 800, "bf16", "bf16", False),
    ("complete", 58, 1600, "f32", "bf16", True),
    ("aer", 96, 960, "f32", "f32", True),                  # streaming, tables in device memory
    ("complete", 68, 700, "bf16", "bf16", True),
])
def test_the_loop_kernels_of_large_layouts(kind, rows, tiles, params, grads, decay):
    """Loops in layouts that take 8 wavefronts, below and above the size from which accesses stream, with the pointer
    tables in the argument block and in device memory: mixing and a step against the same in 64 bits at every element."""
    print("case", kind, rows, tiles, params, grads, decay, flush=True)
    dev, elems = torch.device("cuda:0"), 64 * (8 if params == "bf16" else 4)
    d = tiles * elems - 77
    layout = WL.pack([("a", (d - 2003,)), ("b", (5,)), ("c", (1990,))])
    csr = WL.complete(rows) if kind == "complete" else WL.aer(rows // 4, 0)
    wd = [0.1, 0.0, 0.05] if decay else None
    hp = H.HyperF32(s=1)
    sim = H.GpuSim(rows, rows, layout, hp, [csr], params, grads, weight_decay=wd, pad_fill=777.0)
    assert B.dadam_get_plan_info(sim.h).streaming == (layout.d * rows * 24 > 512 << 20)
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    mask = torch.from_numpy(H.valid_mask(layout)).to(dev)
    lam = torch.from_numpy(H.per_coordinate_decay(layout, wd)).to(dev) if decay else torch.zeros(layout.d, dtype=torch.float64, device=dev)
    g = []
    for i in range(rows):
        sim.x_src[i].copy_(torch.empty(layout.d, device=dev).normal_(0.0, 0.5, generator=gen))
        for t, (lo, hi) in ((sim.m[i], (-1e-3, 1e-3)), (sim.v[i], (3e-5, 1.7e-4))):
            t[mask] = torch.empty(layout.d, device=dev).uniform_(lo, hi, generator=gen)[mask]
        g.append(torch.empty(layout.d, device=dev).normal_(0.0, 1e-2, generator=gen).to(H.TORCH_DT[grads]))
    m0, v0 = [t.clone() for t in sim.m], [t.clone() for t in sim.v]
    tol = 1e-6 if params == "f32" else 1e-2               # float32 sums; one rounding to bfloat16

    def mixed(i):
        want, size = torch.zeros(layout.d, dtype=torch.float64, device=dev), torch.zeros(layout.d, dtype=torch.float64, device=dev)
        for c, w in rows_of_matrix(csr, i):
            want.add_(sim.x_src[c].double(), alpha=w)
            size.add_(sim.x_src[c].double().abs(), alpha=w)
        return want, size

    some = sorted({0, 1, rows // 4, rows // 2, rows - 1})
    sim.mix(0, 0)
    torch.cuda.synchronize()
    first = {i: sim.x_dst[i].clone() for i in some}
    for i in some:
        want, size = mixed(i)
        assert bool(((sim.x_dst[i].double() - want).abs() <= tol * size)[mask].all()), i
        assert bool((sim.x_dst[i][~mask] == 777.0).all()), i
    sim.mix(0, B.DADAM_FORCE_TILE)
    torch.cuda.synchronize()
    if params == "f32":                                     # another order of the same sum: another kernel has run
        assert any(not torch.equal(first[i], sim.x_dst[i]) for i in some)
    f = lambda q: float(np.float32(q))
    b1, b2, lr, eps, t = f(hp.beta1), f(hp.beta2), f(hp.lr), f(hp.eps), 7
    sim.step(g, t, 0, B.DADAM_FUSE_ACCUM)
    torch.cuda.synchronize()
    for i in some:
        want, size = mixed(i)
        gi = g[i].double()
        m, v = b1 * m0[i].double() + (1 - b1) * gi, b2 * v0[i].double() + (1 - b2) * gi * gi
        move = lr * (m / (1 - b1 ** t) / ((v / (1 - b2 ** t)).sqrt() + eps) + lam * sim.x_src[i].double())
        size = size + lr * ((b1 * m0[i].double().abs() + (1 - b1) * gi.abs()) / (1 - b1 ** t) / ((v / (1 - b2 ** t)).sqrt() + eps)
                            + lam * sim.x_src[i].double().abs())
        assert bool(((sim.x_dst[i].double() - (want - move)).abs() <= tol * size)[mask].all()), i
        assert bool(((sim.m[i].double() - m).abs() <= 1e-6 * (b1 * m0[i].double().abs() + (1 - b1) * gi.abs()))[mask].all()), i
        assert bool(((sim.v[i].double() - v).abs() <= 1e-6 * v)[mask].all()), i
        for out in (sim.x_dst[i], sim.m[i], sim.v[i]):
            assert bool((out[~mask] == 777.0).all()), i
    sim.close()


@pytest.mark.parametrize("case", ["loop16-f32", "loop8-f32", "loop8-decay-f32", "loop8-bf16", "tile-decay-f32", "tile-decay-bf16", "foreign-f32"])
def test_a_step_issued_range_by_range_has_the_bits_of_the_whole_one(case):
    """In automatic mode, where the whole step and its ranges are large and small launches: slots of loops (one order of
    the sum for both), and shared rows whose whole step is staged in LDS while its ranges go row by row, with decay; also
    with a row updated in place in the buffer of another row, against the same step out of place."""
    print("case", case, flush=True)
    dtype = "bf16" if "bf16" in case else "f32"
    elems = 64 * (8 if dtype == "bf16" else 4)
    tiles = 210 if "16" in case.split("-")[0] else 700
    n = 12 if not case.startswith("loop") else 24 if "decay" not in case else 60
    sizes = [90 * elems + 7, 200 * elems - 3, 1, (tiles - 400) * elems + 13, 95 * elems] if tiles > 500 else [90 * elems + 7, 61, 60 * elems - 3, 60 * elems]
    layout = WL.pack([(f"t{k}", (s,)) for k, s in enumerate(sizes)])
    wd = [0.1 * (k % 2) for k in range(len(sizes))] if "decay" in case or case.startswith("foreign") else None
    if case.startswith("loop"):
        csr = WL.complete(n)
    elif case.startswith("tile"):
        csr = rows_of_degree(n, 3)
    else:                                                   # only row 0 lists source 1
        col = [[0, 1, 2], [2, 3, 4]] + [[i, 2 if i == n - 1 else i + 1, 0] for i in range(2, n)]
        csr = (np.arange(0, 3 * n + 1, 3, dtype=np.int32), np.array(sum(col, []), np.int32), np.full(3 * n, np.float32(1) / np.float32(3), np.float32))
    sims = [H.GpuSim(n, n, layout, H.HyperF32(s=2), [csr], dtype, dtype, weight_decay=wd) for _ in range(3)]
    for c in range(n):
        x0 = H.to_device(WL.normal_np(700 + c, layout.d, 0.02), dtype, "cuda:0")
        for sim in sims:
            sim.x_src[c].copy_(x0)
    if case.startswith("foreign"):
        for sim in sims[1:]:
            sim.x_dst[0] = sim.x_src[1]
            sim.bind()
    mask = torch.from_numpy(H.valid_mask(layout)).to("cuda:0")
    ranges = [(0, 1), (2, 4), (1, 2), (4, len(sizes))] if len(sizes) > 4 else [(3, 4), (0, 2), (2, 3)]
    for t in range(1, 3 if not case.startswith("foreign") else 2):
        grads = [H.to_device(WL.normal_np(800 + t * 100 + i, layout.d, 1e-3), dtype, "cuda:0") for i in range(n)]
        sims[0].step(grads, t, 0, B.DADAM_FUSE_ACCUM)
        sims[1].step(grads, t, 0, B.DADAM_FUSE_ACCUM)
        for lo, hi in ranges:
            B.dadam_gossip_step_range(sims[2].h, 0, grads, t, B.DADAM_FUSE_ACCUM, lo, hi, sims[2].stream())
        torch.cuda.synchronize()
        for i in range(n):
            for name in ("x_dst", "m", "v", "b"):
                a, whole, parts = (getattr(sim, name)[i][mask] for sim in sims)     # padding is what the buffer held before
                assert torch.equal(a, whole) and torch.equal(a, parts), (t, i, name)
        for sim in sims:
            sim.swap()
    for sim in sims:
        sim.close()


@pytest.mark.parametrize("kind,rows", [("complete", 24), ("aer", 64)])
def test_mixing_with_and_without_the_consensus_error_on_loops(kind, rows):
    """dadam_mix takes the shared sum of a loop, dadam_mix_consensus the listed order: the same within the rounding of a
    float32 sum, and the reported error is that of the sources."""
    print("case", kind, rows, flush=True)
    layout = WL.pack([("a", (70001,)), ("b", (77,))])
    csr = WL.complete(rows) if kind == "complete" else WL.aer(rows // 4, 0)
    sim = H.GpuSim(rows, rows, layout, H.HyperF32(s=1), [csr])
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    for c in range(rows):
        sim.x_src[c].copy_(H.to_device(WL.normal_np(40 + c, layout.d, 0.5), "f32", "cuda:0"))
    sim.mix(0, 0)
    torch.cuda.synchronize()
    plain = [t.clone() for t in sim.x_dst]
    sim.mix_consensus(out)
    torch.cuda.synchronize()
    mask = torch.from_numpy(H.valid_mask(layout)).to("cuda:0")
    for i in range(rows):
        size = sum(w * sim.x_src[c].double().abs() for c, w in rows_of_matrix(csr, i))
        assert bool(((plain[i].double() - sim.x_dst[i].double()).abs() <= 1e-6 * size)[mask].all()), i
    xs = torch.stack([t.double()[mask] for t in sim.x_src])
    want = float((xs - xs.mean(0)).square().sum())
    assert abs(float(out) - want) <= 1e-5 * want           # float32 per element, double sums
    sim.close()
