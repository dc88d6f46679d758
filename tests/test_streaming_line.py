"""Steps of up to three rows around the size from which they stream (344 MB of what they touch): which launches do, without a GPU, and
on the GPU bit for bit against handles over parts of the same elements, which are too small to."""

import pytest
import torch

from paper_2410_11998_amd import binding as B
from paper_2410_11998_amd import workloads as WL

from test_host_abi import _route_answers

import harness as H


def test_steps_of_few_rows_stream_by_what_they_touch(tmp_path):
    """Just below and just above: fused step, update of a range, mixing, accumulation, and what the plan says of the handle.  Sources that no
    row lists, outputs that are sources and elements outside the tensors do not count; the library's answer at 2^20 * 344 bytes exactly."""
    got = _route_answers(tmp_path, "few_rows")
    below, above = "no no no no plan 0", "yes yes no no plan 0"
    assert got.pop("4 rows") == f"{below}, {below}"
    assert len(got) == 9 and set(got.values()) == {f"{below}, {above}"}, got


def test_bench_names_the_kernel_of_steps_that_stream_by_what_they_touch():
    import importlib.util
    import os
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    wl = WL.workload(3)
    for d, streaming, fused in ((12_000_000, 0, "false"), (15_000_000, 0, "true"), (23_000_000, 1, "true")):
        h = B.dadam_init(1, 3, d, [0], [d], B.DADAM_F32, B.DADAM_F32, accum_s=2, device=B.DADAM_DEVICE_NONE)
        info = B.dadam_get_plan_info(h)
        B.dadam_destroy(h)
        assert info.streaming == streaming
        assert bench.kernel_name(info, False, wl, "fused", step_bytes=28 * d) == f"k_direct<TF32,TF32,{fused}>"
        assert bench.kernel_name(info, False, wl, "mix", step_bytes=28 * d) == f"k_direct<TF32,TF32,{'true' if streaming else 'false'}>"


@pytest.mark.gpu
@pytest.mark.parametrize("rows,params,grads", [(1, "f32", "f32"), (1, "bf16", "bf16"), (1, "bf16", "f32"), (2, "f32", "bf16"), (3, "f32", "f32")])
@pytest.mark.parametrize("side", [-4, 4 + 3])
def test_steps_around_the_line(rows, params, grads, side):
    print("case", rows, params, grads, side, flush=True)
    dev = torch.device("cuda:0")
    cols = 3 if rows == 1 else rows
    size = {"f32": 4, "bf16": 2}
    outputs = 0 if rows == 1 else rows                     # the one row is updated in place
    d = (344 << 20) // ((cols + outputs) * size[params] + rows * (size[grads] + 12)) + side
    hp = H.HyperF32(s=2)
    csr = WL.node_share_ring() if rows == 1 else WL.ring(rows)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows * 10 + side)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}

    def draw(n, t, std=1.0):
        return [(torch.randn(d, device=dev, generator=gen) * std).to(t) for _ in range(n)]

    x, g = draw(cols, dt[params]), draw(rows, dt[grads], 1e-2)
    state = [draw(rows, torch.float32, 1e-3), [t.abs() for t in draw(rows, torch.float32, 1e-4)], draw(rows, torch.float32, 1e-3)]
    # parts of less than half the line, ending at multiples of 8 elements (buffers start at multiples of 16 bytes)
    ends = [0] + [d * k // 3 // 8 * 8 for k in (1, 2)] + [d]
    results = []
    for parts in ([(0, d)], list(zip(ends[:-1], ends[1:]))):
        xs = [t.clone() for t in x]
        out = xs[:1] if rows == 1 else [torch.zeros_like(t) for t in xs]
        m, v, b = ([t.clone() for t in s] for s in state)
        for lo, hi in parts:
            cut = lambda ts: [t[lo:hi] for t in ts]  # noqa: E731, B023
            h = B.dadam_init(rows, cols, hi - lo, [0], [hi - lo], H.ABI_DT[params], H.ABI_DT[grads], hp.lr, hp.beta1, hp.beta2, hp.eps, hp.s,
                             device=0)
            B.dadam_set_topology(h, 0, *csr)
            B.dadam_bind(h, cut(xs), cut(out), cut(m), cut(v), cut(b))
            stream = B.current_stream()
            B.dadam_gossip_step(h, 0, cut(g), 3, B.DADAM_FUSE_ACCUM, stream)
            B.dadam_gossip_step(h, 0, cut(g), 4, B.DADAM_FUSE_ACCUM, stream)
            B.dadam_accumulate(h, cut(g), 5, stream)
            B.dadam_mix(h, 0, 0, stream)
            torch.cuda.synchronize()
            B.dadam_destroy(h)
        results.append(xs + out + m + v + b)
    assert all(torch.equal(p, q) for p, q in zip(*results))
    assert not torch.equal(results[0][len(x) + len(x[:1] if rows == 1 else x)], state[0][0])
