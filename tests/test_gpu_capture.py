"""GPU parity of calls recorded into a caller's stream capture.  A replay has to
do the recorded requests on the bytes that the buffers hold then, whatever
calls came between: every form is captured on a context that has no staging
yet, then other requests go through all staging slots (and make them grow)
before each replay, and each replay is compared byte for byte with the CPU
oracle.  Forms: tables among the kernel arguments, tables of one kind beyond
them, both sides in place with predecessor snapshots, tiles with chains (fused
and not), chains alone, more units than are read in place, the call without
allocation (records in kernel arguments, one block of them and several), a
plan, a recorded plan and recorded requests replayed into the capture, and a
request by value."""
import numpy as np
import pytest
import torch

import oracle
from synth import gen, workloads
from tests.gpu_util import ag, device_schedules, first_mismatch

pytestmark = pytest.mark.gpu

ENC, DEC, CTR, ECBE, ECBD = workloads.OP_CBC_ENC, workloads.OP_CBC_DEC, workloads.OP_CTR, 3, 4


def workload(ops, lengths, seed):
    n = len(ops)
    reqs = np.zeros(n, workloads.REQ_DTYPE)
    reqs["length"] = np.asarray(lengths, np.uint64)
    reqs["offset"][1:] = np.cumsum((reqs["length"] + 15) // 16 * 16 + 16)[:-1]
    reqs["op"] = np.asarray(ops, np.uint32)
    reqs["key_idx"] = np.arange(n) % 3
    reqs["iv"] = gen.bytes_(seed, gen.STREAM_IVS, 16 * n).reshape(n, 16)
    keys, kb = workloads.make_keys(seed, 3, [128, 192, 256])
    return workloads.Workload("capture", reqs, keys, kb,
                              int(reqs["offset"][-1] + reqs["length"][-1] + 32), seed)


CASES = {
    "inline": ([CTR] * 8, [4000] * 8),
    "one_kind": ([CTR] * 40, [4096 + 5 * i for i in range(40)]),
    "both_sides": ([DEC, CTR, ECBE, ECBD] * 12, [12288, 5003, 64, 8192] * 12),
    "fused": ([ENC, DEC, CTR] * 20, [320, 12288, 5003] * 20),
    "chains": ([ENC] * 70, [16 * (1 + i % 40) for i in range(70)]),
    "upload": ([CTR, DEC] * 9000, [61, 48] * 9000),
    "one": ([CTR], [70001]),
}


@pytest.mark.parametrize("mode", ["global", "thread_local"])
@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("form,case", [
    ("batch", "inline"), ("single", "one_kind"), ("batch", "both_sides"), ("batch", "fused"),
    ("unfused", "fused"), ("single", "chains"), ("batch", "upload"), ("noalloc", "inline"),
    ("noalloc", "one_kind"), ("noalloc", "both_sides"), ("noalloc", "fused"),
    ("noalloc", "upload"), ("plan", "both_sides"), ("graph", "both_sides"),
    ("requests_graph", "one"), ("request", "one")])
def test_captured_calls(form, case, inplace, mode):
    print(f"[gpu] captured {form}, {case}, inplace={inplace}, {mode}", flush=True)
    a = ag()
    wl = workload(*CASES[case], seed=len(case) + len(form))
    other = workload([CTR, DEC, ENC, ECBE, ECBD] * 60, [9000, 8192, 48, 4096, 16] * 60, seed=7)
    d_s, d_s2 = device_schedules(wl), device_schedules(other)
    inp, inp2 = wl.data(), other.data()
    with a.Context(0) as ctx:
        if form == "unfused":
            ctx.set_config(fuse=0)
        d_in = torch.from_numpy(inp.copy()).cuda()
        d_out = d_in if inplace else torch.from_numpy(workloads.sentinel(inp.size)).cuda()
        o_in = torch.from_numpy(inp2.copy()).cuda()
        o_out = torch.empty_like(o_in)
        r = wl.reqs
        if form in ("plan", "graph"):
            plan = a.Plan(ctx, r, 3, inp.size)
        if form == "graph":
            rec = a.Graph.of_plan(plan, d_s, d_in, d_out)
        elif form == "requests_graph":
            rec = a.Graph.of_requests(ctx, d_s, d_in, d_out, r)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, capture_error_mode=mode):
            if form in ("batch", "unfused"):
                a.batch(ctx, d_s, d_in, d_out, r)
            elif form == "noalloc":
                a.batch_noalloc(ctx, d_s, d_in, d_out, r)
            elif form == "single":
                fn = a.ctr_batch if r["op"][0] == CTR else a.cbc_encrypt_batch
                fn(ctx, d_s, d_in, d_out, r["offset"], r["length"], r["key_idx"], r["iv"])
            elif form == "plan":
                plan.launch(d_s, d_in, d_out)
            elif form == "request":
                a.request_launch(ctx, d_s, d_in, d_out, r[0])
            else:
                rec.launch()
        want = inp.copy() if inplace else workloads.sentinel(inp.size)
        want2 = np.zeros_like(inp2)
        oracle.batch(inp2, want2, other.reqs, other.keys, other.key_bits, n_threads=0)
        touched = np.zeros(inp2.size, bool)
        for q in other.reqs:
            touched[int(q["offset"]):int(q["offset"] + q["length"])] = True
        for k in range(3):
            # Other calls: all staging slots, and the shared array of the
            # no-allocation call.
            for _ in range(5):
                a.batch(ctx, d_s2, o_in, o_out, other.reqs)
            a.batch_noalloc(ctx, d_s2, o_in, o_out, other.reqs[:100 + k])
            src = gen.bytes_(k, 9, inp.size) if k else inp
            d_in.copy_(torch.from_numpy(src.copy()))
            if inplace:
                want = src.copy()
            oracle.batch(src, want, r, wl.keys, wl.key_bits, n_threads=0)
            g.replay()
            torch.cuda.synchronize()
            msg = first_mismatch(d_out.cpu().numpy(), want)
            assert msg is None, f"replay {k}: {msg}"
            msg = first_mismatch(o_out.cpu().numpy()[touched], want2[touched])
            assert msg is None, f"other calls, {k}: {msg}"
        del g
        torch.cuda.synchronize()
        if form in ("graph", "requests_graph"):
            rec.close()
        if form in ("plan", "graph"):
            plan.close()
