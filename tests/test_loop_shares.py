"""Launches in which several workgroups share the rows of a loop's tile, bit for bit against the same step issued tensor by tensor, whose
launches have other numbers of tiles and so of workgroups."""

import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

import harness as H


@pytest.mark.gpu
@pytest.mark.parametrize("kind,rows,tiles,params,grads", [
    ("complete", 17, 128, "f32", "f32"),        # two workgroups of sixteen wavefronts, one row in the second
    ("complete", 33, 85, "f32", "bf16"),        # three
    ("complete", 100, 36, "bf16", "f32"),       # seven, tables in device memory
    ("aer", 96, 42, "f32", "f32"),              # loops of 48, 24 and 24: two, of which the short loops need one and a half
    ("complete", 64, 129, "f32", "f32"),        # one
    ("complete", 32, 2900, "f32", "f32"),       # streaming: one
    ("complete", 96, 4095, "f32", "f32"),       # streaming, the longest launch of two, tables in device memory
    ("complete", 96, 4096, "f32", "f32"),       # one
    ("complete", 97, 768, "bf16", "bf16"),       # two: half of the last round
    ("complete", 97, 769, "bf16", "bf16"),       # one
])
def test_shared_rows_have_the_same_bits(kind, rows, tiles, params, grads):
    print("case", kind, rows, tiles, params, grads, flush=True)
    dev = torch.device("cuda:0")
    d = tiles * 64 * (8 if params == "bf16" else 4) - 6
    sizes = [d // 32 // 8 * 8 + 3, d // 4 // 8 * 8 - 1]
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
    for whole in (True, False):
        out = [torch.full_like(t, 7.0) for t in x]
        state = [t.clone() for t in m + v + b]
        h = B.dadam_init(rows, rows, layout.d, layout.offsets, layout.numels, H.ABI_DT[params], H.ABI_DT[grads], hp.lr, hp.beta1, hp.beta2,
                         hp.eps, hp.s, device=0)
        B.dadam_set_topology(h, 0, *csr)
        B.dadam_bind(h, x, out, state[:rows], state[rows:2 * rows], state[2 * rows:])
        stream = B.current_stream()
        for k in ([(0, 3)] if whole else [(2, 3), (0, 1), (1, 2)]):
            B.dadam_gossip_step_range(h, 0, g, 4, B.DADAM_FUSE_ACCUM, k[0], k[1], stream)
        torch.cuda.synchronize()
        B.dadam_destroy(h)
        results.append(out + state)
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
        err = (results[0][i].double() - (want - hp.lr * u)).abs()
        assert bool((err <= (1e-6 if params == "f32" else 1e-2) * (size + hp.lr * u.abs() + hp.lr))[mask].all())
        assert bool((results[0][i][~mask] == 7.0).all())
