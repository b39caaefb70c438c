"""GPU parity of batches around the size at which the unit table stops being
read from the pinned staging buffer and is uploaded instead (16,384 units), with
more calls in flight than the context has staging slots, on one stream and on
two in turn: each call has its own requests (keys, IVs, order of lengths) and
output, so a table read after its slot was taken again shows."""
import numpy as np
import pytest
import torch

from synth import gen, workloads
from tests.gpu_util import ag, device_schedules, first_mismatch, run_oracle

pytestmark = pytest.mark.gpu

OPS = [workloads.OP_CBC_ENC, workloads.OP_CBC_DEC, workloads.OP_CTR, 3, 4]


def mixed_requests(n_units, seed):
    """Requests of 1 to 3 blocks, one unit each, every operation."""
    r = np.random.default_rng(seed)
    reqs = np.zeros(n_units, workloads.REQ_DTYPE)
    reqs["length"] = 16 * r.integers(1, 4, n_units)
    reqs["offset"] = 64 * np.arange(n_units)
    reqs["op"] = np.asarray(OPS, np.uint32)[r.integers(0, 5, n_units)]
    reqs["key_idx"] = r.integers(0, 3, n_units)
    reqs["iv"] = gen.bytes_(seed, gen.STREAM_IVS, 16 * n_units).reshape(n_units, 16)
    keys, kb = workloads.make_keys(seed, 3, [128, 192, 256])
    return workloads.Workload("unit_tables", reqs, keys, kb, 64 * n_units, seed)


@pytest.mark.parametrize("n_units", [1, 16384, 16385])
@pytest.mark.parametrize("streams", [1, 2])
def test_tables_in_flight(n_units, streams):
    print(f"[gpu] {n_units} units, six calls in flight on {streams} stream(s)", flush=True)
    a = ag()
    ctx = a.Context(0)
    queues = [torch.cuda.Stream() for _ in range(streams)]
    calls = []
    for k in range(6):
        wl = mixed_requests(n_units, 10 * n_units + k)
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
    ctx.close()
