"""The consensus error of large layouts: the kernels that stream and those of sixteen wavefronts, whose lanes are dealt differently
over the sums than in the small ones."""

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

import harness as H

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("rows,dtype", [(4, "f32"),       # two vectors a lane by four wavefronts
                                        (8, "f32"),       # by eight
                                        (17, "f32"),      # by eight, steps by sixteen
                                        (48, "f32"),      # by sixteen
                                        (72, "f32"),      # the same with tables in device memory
                                        (8, "bf16"), (16, "bf16"), (33, "bf16"),
                                        (96, "f32"), (96, "bf16")])      # one vector by sixteen
def test_error_and_mixing_of_layouts_that_stream(rows, dtype, short):
    """The parameters that dadam_mix_consensus leaves are those of dadam_mix bit for bit, padding included, and the error is that of
    64-bit sums over the elements of tensors: what lies between them is NaN in every source.  short: many segments that cut
    tiles, and one long one."""
    print("case", rows, dtype, short, flush=True)
    sizes = [40003, 1, 65536 - 40004 - 40, 32768, 3 * 32768 - 5, 16384 + 2]
    total = (512 << 20) // (24 * rows) // 65536 * 65536 + 2 * 65536 + 3
    if short:
        sizes = [1 + 977 * k % 2300 for k in range(total // 2300)]
    sizes.append(max(total - sum(sizes), 70001))
    layout = WL.pack([("t%d" % k, (n,)) for k, n in enumerate(sizes)])
    sim = H.GpuSim(rows, rows, layout, H.HyperF32(s=1), [WL.static_exponential(rows)], dtype, dtype, pad_fill=777.0)
    assert B.dadam_get_plan_info(sim.h).streaming == 1
    mask = torch.from_numpy(H.valid_mask(layout)).to(DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows)
    noise = lambda std: torch.empty(layout.d, device=DEV).normal_(0.0, std, generator=gen)
    base = noise(0.5)
    for x in sim.x_src:
        x.copy_(base + noise(0.05))
        x[~mask] = float("nan")
    mean = sum(x[mask].double() for x in sim.x_src) / rows
    want = float(sum((x[mask].double() - mean).square().sum() for x in sim.x_src))
    sim.mix()
    torch.cuda.synchronize()
    mixed = [x.clone() for x in sim.x_dst]
    for x in sim.x_dst:
        x[mask] = -1.0
    out = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
    for again in range(2):                  # the second pass finds its partial sums cleared by the first
        sim.mix_consensus(out)
        torch.cuda.synchronize()
        for a, b in zip(mixed, sim.x_dst):
            assert torch.equal(a, b)
        # float32 sums of `rows` squares of distances from source 0, of at most 16 elements a lane, and of 64 lanes; the distances
        # from one source are twice those from the mean, and their squared sum is subtracted: three times the result is added up
        assert abs(float(out.item()) - want) <= 3 * (rows + 16 + 6) * 2.0 ** -24 * want, (again, float(out.item()), want)
    assert all(bool((x[~mask] == 777.0).all()) for x in sim.x_dst)
    sim.close()
