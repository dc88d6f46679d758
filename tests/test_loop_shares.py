"""Launches in which several workgroups share the rows of a loop's tile: how many do, without a GPU, and on the GPU bit for bit against the
same step issued tensor by tensor and mixing by handles over parts, whose launches have other numbers of tiles and so of workgroups."""

import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL
from test_host_abi import _route_answers

import harness as H


def test_streaming_mixing_is_not_shared_out(tmp_path):
    """Handles that stream by their size while their tensors cover few tiles: steps have kernels of shared rows there, mixing has none."""
    shared = {"32": (2, 2), "64": (3, 4), "96": (3, 6)}  # 79 or 40 tiles on 256 compute units; as many as there are rows for sixteen wavefronts
    want = {}
    for rows, by_type in shared.items():
        for dtype, n in zip(("f32", "bf16"), by_type):
            step = f"loop16 shared by {n} streaming"
            want[f"{rows} {dtype}"] = f"{step}, update {step}, mix loop16 shared by 1 streaming"
    assert _route_answers(tmp_path, "sparse_loops") == want


def test_how_many_workgroups_share_a_tile(tmp_path):
    """Fused step, update of the first half, mixing; with one row updated in place always one.  Both sides of each line: a unit for every
    workgroup, as many as have rows, mixing from 32 rows where the tiles divide among 8 dies; streaming steps by their last round."""
    want = {
        "complete16 128 f32": "1 1 1", "complete17 128 f32": "2 2 1", "complete17 129 f32": "1 2 1",
        "complete31 24 f32": "2 2 1", "complete32 24 f32": "2 2 2", "complete33 85 f32": "3 3 1", "complete33 86 f32": "2 3 1",
        "complete64 64 bf16": "4 4 4", "complete64 129 f32": "1 4 1", "complete96 42 f32": "6 6 1", "complete96 40 bf16": "6 6 6",
        "complete100 36 bf16": "7 7 1", "halves96 16 f32": "3 3 3", "halves96 42 f32": "2 3 1", "halves96 43 f32": "1 3 1",
        # streaming: no mixing; one loop of 96 rows and more
        "complete32 2900 f32": "1 1 1", "complete95 1100 f32": "1 1 1", "halves128 900 f32": "1 1 1",
        # a round of 768 tiles in float32: a quarter of one more, half a round where a tile is cut, up to 2048 tiles
        "complete128 768 f32": "1 1 1", "complete128 769 f32 whole": "2 1 1", "complete128 960 f32 whole": "2 1 1", "complete128 961 f32 whole": "1 1 1",
        "complete128 961 f32": "2 1 1", "complete128 1152 f32": "2 1 1", "complete128 1153 f32": "1 1 1", "complete96 1536 f32": "1 1 1",
        "complete96 1537 f32": "2 1 1", "complete96 1728 f32": "2 2 1", "complete96 1729 f32": "1 2 1", "complete96 2305 f32": "1 1 1",
        # of 512 in bfloat16
        "complete97 512 bf16": "1 1 1", "complete97 513 bf16 whole": "2 1 1", "complete97 640 bf16 whole": "2 1 1", "complete97 641 bf16 whole": "1 1 1",
        "complete97 768 bf16": "2 1 1", "complete97 769 bf16": "1 1 1", "complete97 1024 bf16": "1 1 1", "complete97 1152 bf16": "2 2 1",
        "complete97 1153 bf16": "1 2 1", "complete97 1664 bf16 whole": "2 1 1", "complete97 2049 bf16 whole": "1 1 1",
    }
    got = _route_answers(tmp_path, "loop_shares")
    # up to 16384 wavefronts count as a small launch, whose lanes all search the segments: shared workgroups are in the count
    assert got.pop("wide search, 1030") == "2 no" and got.pop("wide search, 1300") == "1 yes"
    assert got == {k: v + " | 1 1" for k, v in want.items()}


@pytest.mark.gpu
@pytest.mark.parametrize("rows,dtype", [(32, "f32"), (64, "bf16"), (96, "f32"), (96, "bf16")])
@pytest.mark.parametrize("tensors", [1, 12])
def test_mixing_of_few_tiles_in_a_handle_that_streams(rows, dtype, tensors):
    """20000 elements in the middle of 2.3e7 of all rows, as one tensor or as twelve short ones (which have a map), on the complete graph: every
    row gets the mean of the sources, mixing and steps keep to the tensors."""
    print("case", rows, dtype, tensors, flush=True)
    dev = torch.device("cuda:0")
    d = 23000000 // rows // 8 * 8 + 8
    lead, each = d // 2 // 8 * 8, 20000 // tensors
    offsets = [lead + k * (-(-each // 8) * 8) for k in range(tensors)] + [d]
    numels = [each] * tensors + [0]
    inside = torch.zeros(d, dtype=torch.bool, device=dev)
    for o, n in zip(offsets, numels):
        inside[o:o + n] = True
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows)
    dt = H.TORCH_DT[dtype]
    # eighths between -1 and 1
    x = [torch.full((d,), float("nan"), dtype=dt, device=dev) for _ in range(rows)]
    for t in x:
        t[inside] = (torch.randint(-8, 9, (int(inside.sum()),), device=dev, generator=gen).float() / 8).to(dt)
    out = [torch.full_like(t, 7.0) for t in x]
    g = [torch.zeros_like(t) for t in x]
    state = [torch.full((d,), 0.0, device=dev) for _ in range(3 * rows)]
    h = B.dadam_init(rows, rows, d, offsets, numels, H.ABI_DT[dtype], H.ABI_DT[dtype], 1e-3, 0.9, 0.999, 1e-8, 2, device=0)
    assert B.dadam_get_plan_info(h).streaming == 1
    B.dadam_set_topology(h, 0, *WL.complete(rows))
    B.dadam_bind(h, x, out, state[:rows], state[rows:2 * rows], state[2 * rows:])
    stream = B.current_stream()
    want = sum(t[inside].double() for t in x) / rows
    # partial sums are at most 1: a rounding of 2^-25 for the weights together and for each term and part, and that of the result
    bound = 2 * rows * 2.0 ** -25 + (want.abs() * 2.0 ** -8 if dtype == "bf16" else 0.0)
    for call in (lambda: B.dadam_mix(h, 0, 0, stream), lambda: B.dadam_gossip_step(h, 0, g, 1, B.DADAM_FUSE_ACCUM, stream),
                 lambda: B.dadam_gossip_step(h, 0, g, 1, 0, stream)):
        for t in out:
            t.fill_(7.0)
        call()
        torch.cuda.synchronize()
        for t in out:
            assert bool(((t[inside].double() - want).abs() <= bound).all())
            assert bool((t[~inside] == 7.0).all())
    B.dadam_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,rows,tiles,params,grads", [
    ("complete", 17, 128, "f32", "f32"),        # two workgroups of sixteen wavefronts, one row in the second
    ("complete", 33, 85, "f32", "bf16"),        # three
    ("complete", 64, 24, "f32", "f32"),         # four, in mixing too
    ("complete", 100, 36, "bf16", "f32"),       # seven, tables in device memory
    ("complete", 100, 32, "bf16", "bf16"),      # seven, in mixing too
    ("aer", 96, 42, "f32", "f32"),              # loops of 48, 24 and 24: two, of which the short loops need one and a half
    ("complete", 64, 129, "f32", "f32"),        # one
    ("complete", 32, 2900, "f32", "f32"),       # streaming: one
    ("complete", 96, 1728, "f32", "f32"),       # streaming, the longest launch of two, tables in device memory
    ("complete", 96, 1729, "f32", "f32"),       # one
    ("complete", 96, 4095, "f32", "f32"),       # one, long
    ("complete", 96, 4096, "f32", "f32"),
    ("complete", 97, 768, "bf16", "bf16"),      # two: half of the last round, a tile is cut
    ("complete", 97, 769, "bf16", "bf16"),      # one
])
def test_shared_rows_have_the_same_bits(kind, rows, tiles, params, grads):
    for gaps in (True, False):                  # with gaps of a few elements small layouts have a map
        same_bits(kind, rows, tiles, params, grads, gaps)


def same_bits(kind, rows, tiles, params, grads, gaps):
    print("case", kind, rows, tiles, params, grads, gaps, flush=True)
    dev = torch.device("cuda:0")
    d = tiles * 64 * (8 if params == "bf16" else 4) - 6
    sizes = [d // 32 // 8 * 8 + 3, d // 4 // 8 * 8 - 1] if gaps else [d // 32 // 8 * 8, d // 4 // 8 * 8]
    layout = WL.pack([("t%d" % k, (n,)) for k, n in enumerate(sizes + [d - sum(-(-n // 8) * 8 for n in sizes)])])
    assert -(-layout.d // (64 * (8 if params == "bf16" else 4))) == tiles
    csr = WL.complete(rows) if kind == "complete" else WL.aer(rows // 4, 0)
    hp = H.HyperF32(s=2)
    gen = torch.Generator(device=dev)
    gen.manual_seed(tiles)

    def draw(dt, std, low=None):
        return [(torch.empty(layout.d, device=dev).normal_(0.0, std, generator=gen) if low is None else
                 torch.empty(layout.d, device=dev).uniform_(low, std, generator=gen)).to(dt) for _ in range(rows)]

    x, g = draw(H.TORCH_DT[params], 0.5), draw(H.TORCH_DT[grads], 1e-2)
    m, v, b = draw(torch.float32, 1e-3), draw(torch.float32, 1e-4, 1e-5), draw(torch.float32, 1e-3)
    results = []

    def handle(lo, hi, offsets, numels, out, state):
        cut = lambda ts: [t[lo:hi] for t in ts]  # noqa: E731
        h = B.dadam_init(rows, rows, hi - lo, offsets, numels, H.ABI_DT[params], H.ABI_DT[grads], hp.lr, hp.beta1, hp.beta2, hp.eps, hp.s, device=0)
        B.dadam_set_topology(h, 0, *csr)
        B.dadam_bind(h, cut(x), cut(out), cut(state[:rows]), cut(state[rows:2 * rows]), cut(state[2 * rows:]))
        return h

    stream = B.current_stream()
    for whole in (True, False):
        out, updated, mixed = ([torch.full_like(t, 7.0) for t in x] for _ in range(3))
        state = [t.clone() for t in m + v + b]
        for to, flags in ((out, B.DADAM_FUSE_ACCUM), (updated, 0)):
            h = handle(0, layout.d, layout.offsets, layout.numels, to, state)
            for k in ([(0, 3)] if whole else [(2, 3), (0, 1), (1, 2)]):
                B.dadam_gossip_step_range(h, 0, g, 4, flags, k[0], k[1], stream)
            torch.cuda.synchronize()
            B.dadam_destroy(h)
        # the parts of a layout of more than 512 tiles may have another kernel, which sums in another order
        ends = [0, layout.d] if whole or tiles > 512 else [0, int(layout.offsets[1]), layout.d // 2 // 8 * 8, layout.d]
        for lo, hi in zip(ends[:-1], ends[1:]):
            inside = [(max(int(o), lo), min(int(o) + int(n), hi)) for o, n in zip(layout.offsets, layout.numels)]
            inside = [(p, q) for p, q in inside if p < q]
            h = handle(lo, hi, [p - lo for p, _ in inside], [q - p for p, q in inside], mixed, state)
            B.dadam_mix(h, 0, 0, stream)
            torch.cuda.synchronize()
            B.dadam_destroy(h)
        results.append(out + updated + mixed + state)
    assert all(torch.equal(p, q) for p, q in zip(*results))
    # against 64 bits, two rows: the mean of what is within the row's loop, less the step
    mask = torch.from_numpy(H.valid_mask(layout)).to(dev)
    for i in (0, rows - 1):
        cols = [int(c) for c in csr[1][csr[0][i]:csr[0][i + 1]]]
        want = sum(x[c].double() for c in cols) / len(cols)
        size = sum(x[c].double().abs() for c in cols) / len(cols)
        gd = g[i].double()
        c1, c2 = 1 - hp.beta1 ** 2, 1 - hp.beta2 ** 2
        u = ((hp.beta1 * m[i].double() + (1 - hp.beta1) * gd) / c1) / (((hp.beta2 * v[i].double() + (1 - hp.beta2) * gd * gd) / c2).sqrt() + hp.eps)
        err = (results[0][2 * rows + i].double() - want).abs()
        # a rounding of 2^-24 of the sum's size for each source and its weight, and in bfloat16 that of the result
        assert bool((err <= 2 * rows * 2.0 ** -24 * size + (2.0 ** -8 * want.abs() if params == "bf16" else 0.0))[mask].all())
        err = (results[0][i].double() - (want - hp.lr * u)).abs()
        assert bool((err <= (1e-6 if params == "f32" else 1e-2) * (size + hp.lr * u.abs() + hp.lr))[mask].all())
        assert bool((results[0][i][~mask] == 7.0).all())
