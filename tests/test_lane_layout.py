"""Where the lanes of the streaming kernels lie over the elements: on the CPU from the kernel source's own text, and on the GPU
bit for bit against handles small enough to take the kernels whose lanes lie side by side."""

import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import build as bld
from paper_2410_11998_amd import workloads as WL

import harness as H


def test_every_element_has_one_lane(tmp_path):
    clang = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")
    if clang is None:
        pytest.skip("no clang++")
    src = open(os.path.join(bld.CSRC, "dadam_device.h")).read()
    cut = lambda a, b: src[src.index(a):src.index(b, src.index(a))]
    (tmp_path / "layout.inc").write_text(cut("template <bool STREAM>\nconstexpr int kGroupStep", "typedef float f4")
                                         + cut("__device__ __forceinline__ uint32_t die_block_order", "// Direct mode with a sharing order")
                                         + cut("__device__ __forceinline__ bool die_block_piece", "// Where a lane's first group")
                                         + cut("template <int VEC, int U, bool STREAM>", "// One step of the search of all lanes"))
    exe = str(tmp_path / "layout")
    subprocess.run([clang, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I", str(tmp_path),
                    os.path.join(os.path.dirname(os.path.abspath(__file__)), "emulate_lane_layout.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.count(": right") == 9, (r.stdout, r.stderr[-2000:])


def test_groups_at_the_edges_of_a_range(tmp_path):
    clang = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")
    if clang is None:
        pytest.skip("no clang++")
    src = open(os.path.join(bld.CSRC, "dadam_device.h")).read()
    b = src.index("// Algorithm 3, lines 6-13, for one element.")
    (tmp_path / "helpers.inc").write_text(src[src.index("typedef float f4 __attribute__"):src.rindex("// ----", 0, b)])
    a = src.index("template <typename A>\n__device__ __forceinline__ int clip_of")
    (tmp_path / "clip.inc").write_text(src[a:src.index("// Pointers of the bound buffers.", a)])
    exe = str(tmp_path / "clip")
    subprocess.run([clang, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I", str(tmp_path),
                    os.path.join(os.path.dirname(os.path.abspath(__file__)), "emulate_group_clip.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "bad 0, tiles by groups many, by elements some\n", (r.stdout, r.stderr[-2000:])


@pytest.mark.gpu
@pytest.mark.parametrize("rows,deg,tiles,dtype", [(18, 2, 1024, "f32"), (26, 2, 1100, "bf16"), (100, 3, 1027, "f32"), (65, 2, 1500, "f32")])
def test_rows_walked_in_runs_give_the_tile_kernels_bits(rows, deg, tiles, dtype):
    """Launches of 1024 tiles and more that do not stream: a die walks runs of pieces row after row, the last run shorter,
    dies with a piece fewer; a step of every phase against the tile kernel, with decay and ragged ends."""
    print("case", rows, deg, tiles, dtype, flush=True)
    elems = 64 * (8 if dtype == "bf16" else 4)
    layout = WL.pack([("a", (900 * elems + 13,)), ("b", (5,)), ("c", ((tiles - 901) * elems - 40,))])
    w = np.float32(1.0) / np.float32(deg)
    csr = (np.arange(0, rows * deg + 1, deg, dtype=np.int32), np.array([(i + k) % rows for i in range(rows) for k in range(deg)], np.int32),
           np.full(rows * deg, w, np.float32))
    sims = [H.GpuSim(rows, rows, layout, H.HyperF32(s=2), [csr], dtype, dtype, weight_decay=[0.1, 0.0, 0.05], pad_fill=777.0) for _ in range(2)]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    for c in range(rows):
        sims[0].x_src[c].normal_(0.0, 0.02, generator=gen)
        sims[1].x_src[c].copy_(sims[0].x_src[c])
    for t, flags in ((1, B.DADAM_FUSE_ACCUM), (2, B.DADAM_FUSE_ACCUM), (3, 0)):
        grads = [torch.empty(layout.d, device="cuda:0").normal_(0.0, 1e-2, generator=gen).to(H.TORCH_DT[dtype]) for _ in range(rows)]
        for sim, mode in zip(sims, (0, B.DADAM_FORCE_TILE)):
            sim.step(grads, t, 0, flags | mode)
        torch.cuda.synchronize()
        for i in range(rows):
            for name in ("x_dst", "m", "v", "b"):
                assert torch.equal(getattr(sims[0], name)[i], getattr(sims[1], name)[i]), (t, i, name)
        for sim in sims:
            sim.swap()
    for sim in sims:
        sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows,topology,params,grads,decay", [
    (4, "ring", "f32", "f32", True),            # tile kernel, two vectors by 4, 8, 16 wavefronts
    (8, "ring", "f32", "bf16", False),
    (17, "exp", "f32", "f32", True),
    (72, "ring", "f32", "f32", False),          # pointer tables in device memory
    (8, "exp", "bf16", "bf16", True),
    (1, "share", "f32", "f32", True),           # direct kernel, nothing shared
    (1, "share", "bf16", "bf16", False),
    (32, "one_peer", "f32", "f32", False),      # direct kernel, rows in groups per die, mixing by whole items
    (64, "one_peer", "bf16", "f32", True),
    (40, "one_peer", "f32", "f32", True),
    (18, "one_peer", "bf16", "bf16", True),     # runs of pieces row after row
    (33, "ring", "f32", "f32", True),
    (96, "exp", "f32", "f32", True),            # tile of sixteen wavefronts, one workgroup to a compute unit
    (96, "exp", "bf16", "bf16", False),
])
def test_streaming_kernels_give_the_bits_of_small_handles(rows, topology, params, grads, decay):
    """A layout that streams, cut into tensors at and beside the edges of tiles and blocks; the same buffers, piece by piece,
    through handles that do not stream.  Every phase, mixing, and accumulation by itself."""
    print("case", rows, topology, params, grads, decay, flush=True)
    dev = torch.device("cuda:0")
    share = topology == "share"
    cols = 3 if share else rows
    chunk = (512 << 20) // (24 * rows) // 65536 * 65536          # the largest piece that does not stream, less than a block
    sizes = [40003, 1, 65536 - 40004 - 40, 32768, 3 * 32768 - 5, 16384 + 2]
    sizes.append(max(chunk + 70001, 8 * 65536) - sum(sizes))       # and long segments on average
    layout = WL.pack([("t%d" % k, (n,)) for k, n in enumerate(sizes)])
    wd = [0.1 * (k % 2) for k in range(len(sizes))] if decay else None
    csr = {"ring": lambda: WL.ring(rows), "exp": lambda: WL.static_exponential(rows), "share": WL.node_share_ring,
           "one_peer": lambda: WL.one_peer_exponential(rows, 1)}[topology]()
    hp = H.HyperF32(s=2)
    sims = [H.GpuSim(rows, cols, layout, hp, [csr], params, grads, weight_decay=wd, inplace=share, pad_fill=777.0) for _ in range(2)]
    big, ref = sims
    assert B.dadam_get_plan_info(big.h).streaming == 1
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    mask = torch.from_numpy(H.valid_mask(layout)).to(dev)
    noise = lambda std: torch.empty(layout.d, device=dev).normal_(0.0, std, generator=gen)
    for c in range(cols):
        x = noise(0.5)
        for sim in sims:
            sim.x_src[c][mask] = x.to(sim.x_src[c].dtype)[mask]
    grad = [noise(1e-2).to(H.TORCH_DT[grads]) for _ in range(rows)]
    # handles over [0, chunk), [chunk, 2 chunk), ... of the reference's buffers
    xdt, gdt = [B.DADAM_BF16 if t == "bf16" else B.DADAM_F32 for t in (params, grads)]
    small = []
    for lo, hi in [(k, min(k + chunk, layout.d)) for k in range(0, layout.d, chunk)]:
        parts = [(max(int(o), lo), min(int(o) + int(n), hi), 0.0 if wd is None else wd[k])
                 for k, (o, n) in enumerate(zip(layout.offsets, layout.numels)) if int(o) < hi and int(o) + int(n) > lo]
        h = B.dadam_init(rows, cols, hi - lo, [a - lo for a, _, _ in parts], [b - a for a, b, _ in parts], xdt, gdt, hp.lr, hp.beta1,
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
    if not share:
        big.mix(0, 0)
        on_small(lambda h, g: B.dadam_mix(h, 0, 0, stream))
        same("mix")
    B.dadam_gossip_step_range(big.h, 0, grad, 4, B.DADAM_FUSE_ACCUM, 0, 3, stream)       # a block cut by the range, and the rest
    B.dadam_gossip_step_range(big.h, 0, grad, 4, B.DADAM_FUSE_ACCUM, 3, len(sizes), stream)
    on_small(lambda h, g: B.dadam_gossip_step(h, 0, g, 4, B.DADAM_FUSE_ACCUM, stream))
    same("ranges")
    for h, _, _ in small:
        B.dadam_destroy(h)
    for sim in sims:
        sim.close()
