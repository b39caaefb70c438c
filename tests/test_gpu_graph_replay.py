"""GPU parity of recorded launches (aes_plan_graph, aes_requests_graph): four
requests (replayed as launches) and five (a HIP graph), zero-length ones among
them, and plans of one kernel, of several, in place with several tiles per
request, and fused; each replayed three times with the program's own work and
a changed launch configuration of the context between the replays, every
replay byte for byte against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from synth import gen, workloads
from tests.gpu_util import ag, device_schedules, first_mismatch

pytestmark = pytest.mark.gpu


def requests(ops, lengths, seed):
    n = len(ops)
    reqs = np.zeros(n, workloads.REQ_DTYPE)
    reqs["length"] = np.asarray(lengths, np.uint64)
    reqs["offset"][1:] = np.cumsum(reqs["length"] + 16)[:-1]
    reqs["op"] = np.asarray(ops, np.uint32)
    reqs["key_idx"] = np.arange(n) % 3
    reqs["iv"] = gen.bytes_(seed, gen.STREAM_IVS, 16 * n).reshape(n, 16)
    keys, kb = workloads.make_keys(seed, 3, [128, 192, 256])
    return workloads.Workload("graph", reqs, keys, kb,
                              int(reqs["offset"][-1] + reqs["length"][-1] + 16), seed)


ENC, DEC, CTR = workloads.OP_CBC_ENC, workloads.OP_CBC_DEC, workloads.OP_CTR


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("what,ops,lengths", [
    ("requests", [CTR, DEC, ENC, 3, CTR], [5008, 20000, 320, 4096, 0]),  # four with bytes
    ("requests", [CTR, DEC, ENC, 3, 4], [5008, 20000, 320, 4096, 64]),
    ("plan", [DEC] * 6, [4096, 20000, 16, 8192, 12288, 65536]),
    ("plan", [DEC, CTR, 3, 4] * 4, [12288, 5008, 64, 8192] * 4),
    ("plan", [DEC, CTR, ENC, 4] * 4, [12288, 5008, 64, 8192] * 4)])
def test_replays(what, ops, lengths, inplace):
    print(f"[gpu] {what} graph of {len(ops)} requests, inplace={inplace}", flush=True)
    a = ag()
    wl = requests(ops, lengths, len(ops) + len(what))
    d_s = device_schedules(wl)
    inp = wl.data()
    with a.Context(0) as ctx:
        d_in = torch.from_numpy(inp.copy()).cuda()
        d_out = d_in if inplace else torch.from_numpy(workloads.sentinel(inp.size)).cuda()
        if what == "plan":
            plan = a.Plan(ctx, wl.reqs, 3, inp.size)
            g = a.Graph.of_plan(plan, d_s, d_in, d_out)
        else:
            g = a.Graph.of_requests(ctx, d_s, d_in, d_out, wl.reqs)
        want = inp.copy() if inplace else workloads.sentinel(inp.size)
        for k in range(3):
            src = inp if not inplace else want.copy()
            oracle.batch(src, want, wl.reqs, wl.keys, wl.key_bits, n_threads=0)
            g.launch()
            torch.cuda.synchronize()
            msg = first_mismatch(d_out.cpu().numpy(), want)
            assert msg is None, f"replay {k}: {msg}"
            ctx.set_config(tile_bytes=1024 << k, ctr_nb=1, dec_nb=1, fuse=k & 1, grid=3 + k)
            scratch = torch.full((1 << 20,), k, dtype=torch.uint8, device="cuda")
            assert int(scratch.sum()) == k << 20
        g.close()
        if what == "plan":
            plan.close()
