"""Links loaded again into a context reach every later call: eager ones in both layouts
and storages, and replays of a graph that was captured before.  Where memory does not
hold both layouts, the calls run on the plane layout alone."""
import numpy as np
import pytest
import torch

import oracle

from gpu_util import DEV, context, elem_rel_err, emulated_sloppy_apply, inputs, site_scaled_err, to_dev
from test_gpu_operator import SLOPPY_TOL

pytestmark = pytest.mark.gpu


# one column on any lattice and two to four above 8192 sites of a parity run on the planes
@pytest.mark.parametrize("dims,n", [((4, 4, 4, 6), 1), ((4, 4, 4, 6), 5), ((16, 16, 12, 6), 3)])
def test_reloaded_links_reach_eager_calls(dims, n):
    ctx = None
    for seed in (21100, 21200, 21300):
        fat, lng, B = inputs(dims, True, n, seed)
        if ctx is None:
            ctx = context(dims, True, fat, lng, 0.07)
        else:
            ctx.load_links(fat, lng)
        op = oracle.Operator(dims, fat, lng, 0.07)
        x = to_dev(B)
        # the tolerances of the operator tests
        assert elem_rel_err(ctx.apply(x).cpu().numpy(), op.apply(B)).max() <= 1e-12
        for prec in ("fp32", "fix16"):
            got = ctx.apply_prec(prec, x).cpu().numpy()
            assert site_scaled_err(got, emulated_sloppy_apply(op, prec, B)) <= SLOPPY_TOL[prec]


@pytest.mark.parametrize("eager_first", [True, False])
@pytest.mark.parametrize("dims,n", [((4, 4, 4, 6), 1), ((4, 4, 4, 6), 5), ((16, 16, 12, 6), 3)])
def test_graph_replays_see_reloaded_links(dims, n, eager_first):
    """A captured bcg_apply_noalloc replays with the links loaded last, whether or not an
    eager call came before the capture."""
    fat, lng, B = inputs(dims, True, n, 21500)
    stream = torch.cuda.Stream(DEV)
    with torch.cuda.stream(stream):
        ctx = context(dims, True, fat, lng, 0.07)
        x = to_dev(B)
        out = torch.empty_like(x)
        if eager_first:
            ctx.apply(x)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.apply_noalloc(x, out)
        for seed in (21500, 21600, 21700):
            fat, lng, _ = inputs(dims, True, 1, seed)
            ctx.load_links(fat, lng)
            ref = oracle.Operator(dims, fat, lng, 0.07).apply(B)
            for _ in range(3):
                out.fill_(float("nan"))
                graph.replay()
                stream.synchronize()
                assert elem_rel_err(out.cpu().numpy(), ref).max() <= 1e-12
                assert torch.equal(ctx.apply(x), out)


def test_links_in_one_layout_where_memory_is_short():
    """A context above 349525 sites of a parity takes the row layout's copy of the links
    (1.8 GB here) only beside four times as much free memory, and gives it back to a call
    whose workspace (3.6 GB for 64 columns) does not fit otherwise."""
    dims = (32, 32, 32, 24)
    vh = 32 * 32 * 32 * 12
    copy = 2 * 16 * 9 * vh * 16
    fat, lng, _ = inputs(dims, True, 1, 21800)
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.view_as_complex(torch.randn(64, vh, 3, 2, dtype=torch.float64, device=DEV, generator=g))
    out = torch.empty_like(x)

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info(DEV)[0]

    def hold(left):
        """Takes what is free but for about `left` bytes."""
        blocks = []
        while (n := min(free() - left, 16 << 30)) > 64 << 20:
            blocks.append(torch.empty(n, dtype=torch.uint8, device=DEV))
        return blocks

    def rel(a, b):
        return float((a - b).abs().max() / b.abs().max())

    ctx = context(dims, True, fat, lng, 0.07)
    ref = ctx.apply(x[:8]).clone()
    one = ctx.apply(x[:1]).clone()
    assert rel(one, ref[:1]) <= 1e-12
    blocks = hold(2500 << 20)
    ctx.apply(x, out)  # in place of the row copy
    assert rel(out[:8], ref) <= 1e-12
    assert torch.equal(ctx.apply(x[:8]), out[:8])  # the same kernels now
    del blocks
    blocks = hold(4500 << 20)
    before = free()
    short = context(dims, True, fat, lng, 0.07)  # planes 1.8, staging 0.9 GB
    assert before - free() < 1.5 * copy
    for n in (1, 8):
        assert rel(short.apply(x[:n]), ref[:n]) <= 1e-12
    del blocks
    short.close()
    free()
    ctx.load_links(fat, lng)  # room again: both layouts
    assert torch.equal(ctx.apply(x[:8]), ref)
    ctx.close()
