"""GPU parity of routes for small and middling calls, byte for byte against the
CPU oracle: the call without allocation with its units among the kernel
arguments, and with tables that its tile kernels claim from (counters cleared
by the call, on both sides and on a packed grid); tables of one kind just over
the kernel arguments with more calls in flight than there are staging slots;
and the default tile shape under a set grid, which keeps the tile kernels, with
fewer units than a workgroup has waves."""
import numpy as np
import pytest
import torch

from synth import workloads
from tests.gpu_util import ag, device_schedules, first_mismatch, run_gpu, run_oracle
from tests.test_gpu_short_tiles import OPS, requests

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    c = ag().Context(0)
    yield c
    c.close()


def noalloc(ctx, wl, inplace):
    inp = wl.data()
    d_in = torch.from_numpy(inp.copy()).cuda()
    d_out = d_in if inplace else torch.from_numpy(workloads.sentinel(inp.size)).cuda()
    ag().batch_noalloc(ctx, device_schedules(wl), d_in, d_out, wl.reqs)
    torch.cuda.synchronize()
    msg = first_mismatch(d_out.cpu().numpy(), run_oracle(wl, inp, inplace=inplace))
    assert msg is None, msg


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n", [1, 31, 32, 33])
def test_noalloc_units_among_arguments(ctx, op, n, inplace):
    print(f"[gpu] noalloc, {n} units of {op}, inplace={inplace}", flush=True)
    for seed in (n, n + 100):
        lengths = np.random.default_rng(seed).integers(1, 257, n) * 16
        if op == "ctr":
            lengths[-1] -= 7
        noalloc(ctx, requests(op, lengths, seed), inplace)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("grid", [0, 200, 3072])
def test_noalloc_counters(ctx, grid, inplace):
    """Both tile kernels in one call, beyond what the kernels for short launches
    take, three calls in a row of falling size."""
    print(f"[gpu] noalloc, both sides, grid={grid}, inplace={inplace}", flush=True)
    ctx.set_config(grid=grid, fuse=0)
    for n in (7001, 5000, 3333):
        wl = requests("ctr", [4096] * (2 * n), n)
        wl.reqs["op"][::2] = workloads.OP_CBC_DEC
        noalloc(ctx, wl, inplace)


@pytest.mark.parametrize("streams", [1, 2])
@pytest.mark.parametrize("op", ["ctr", "cbc_dec", "cbc_enc"])
@pytest.mark.parametrize("n", [33, 200])
def test_tables_of_one_kind_in_flight(ctx, op, n, streams):
    print(f"[gpu] {n} units of {op}, six calls on {streams} stream(s)", flush=True)
    a = ag()
    queues = [torch.cuda.Stream() for _ in range(streams)]
    calls = []
    for k in range(6):
        wl = requests("ctr" if op == "cbc_enc" else op,
                      np.random.default_rng(n + k).integers(1, 65, n) * 16, n + k)
        if op == "cbc_enc":
            wl.reqs["op"] = workloads.OP_CBC_ENC
        inp = wl.data()
        calls.append((wl, inp, device_schedules(wl), torch.from_numpy(inp).cuda(),
                      torch.from_numpy(workloads.sentinel(inp.size)).cuda()))
    torch.cuda.synchronize()
    for k, (wl, _, scheds, d_in, d_out) in enumerate(calls):
        with torch.cuda.stream(queues[k % streams]):
            a.batch(ctx, scheds, d_in, d_out, wl.reqs)
    torch.cuda.synchronize()
    for k, (wl, inp, _, _, d_out) in enumerate(calls):
        msg = first_mismatch(d_out.cpu().numpy(), run_oracle(wl, inp))
        assert msg is None, f"call {k}: {msg}"


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n,grid", [(1, 256), (5, 256), (15, 1), (17, 1), (300, 256), (300, 19)])
def test_default_shape_on_a_set_grid(ctx, op, n, grid, inplace):
    print(f"[gpu] {n} units of {op} on {grid} workgroups, inplace={inplace}", flush=True)
    ctx.set_config(grid=grid)
    lengths = np.random.default_rng(n).integers(1, 129, n) * 16
    if op == "ctr":
        lengths[-1] -= 3
    wl = requests(op, lengths, n)
    inp = wl.data()
    want = run_oracle(wl, inp, inplace=inplace)
    for form in ("plan", "batch"):
        msg = first_mismatch(run_gpu(ctx, wl, inp, form=form, inplace=inplace), want)
        assert msg is None, f"{form}: {msg}"
