"""GPU parity of buffers whose base is not 16-byte aligned (views into larger
tensors), in every form and for launches of all sizes, byte for byte against
the CPU oracle: no alignment of d_in and d_out is asked for, only offsets in
them are multiples of 16."""
import numpy as np
import pytest
import torch

from synth import workloads
from tests.gpu_util import ag, device_schedules, first_mismatch, run_oracle
from tests.test_gpu_short_tiles import OPS, requests

pytestmark = pytest.mark.gpu

SIZES = {"few": [4096, 16, 1040, 33 * 16], "one_pass": [4096] * 300 + [48],
         "small": [16 * (1 + i % 64) for i in range(6000)],
         "uneven": [16 * (1 + (i * i) % 200) if i % 3 else 64 for i in range(7000)],
         "multi_tile": [12288 + 16 * i for i in range(40)]}


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS) + ["cbc_enc"])
@pytest.mark.parametrize("size", list(SIZES))
def test_bases(size, op, inplace):
    print(f"[gpu] misaligned bases: {op}, {size}, inplace={inplace}", flush=True)
    a = ag()
    wl = requests("ctr" if op == "cbc_enc" else op, SIZES[size], len(size))
    if op == "cbc_enc":
        wl.reqs["op"] = workloads.OP_CBC_ENC
    if op == "ctr":
        wl.reqs["length"][::7] -= 3
    inp = wl.data()
    want = run_oracle(wl, inp, inplace=inplace)
    d_s = device_schedules(wl)
    with a.Context(0) as ctx:
        plan = a.Plan(ctx, wl.reqs, 3, inp.size)
        for shift_in, shift_out in ((1, 0), (0, 2), (4, 8), (15, 1)):
            d_in = torch.empty(inp.size + 16, dtype=torch.uint8, device="cuda")
            d_in = d_in[shift_in:shift_in + inp.size]
            for form in ("batch", "plan", "noalloc", "request"):
                d_in.copy_(torch.from_numpy(inp.copy()))
                d_out = d_in
                if not inplace:
                    d_out = torch.empty(inp.size + 16, dtype=torch.uint8, device="cuda")
                    d_out = d_out[shift_out:shift_out + inp.size]
                    d_out.copy_(torch.from_numpy(workloads.sentinel(inp.size)))
                assert d_in.data_ptr() % 16 == shift_in
                if form == "batch":
                    a.batch(ctx, d_s, d_in, d_out, wl.reqs)
                elif form == "plan":
                    plan.launch(d_s, d_in, d_out)
                elif form == "noalloc":
                    a.batch_noalloc(ctx, d_s, d_in, d_out, wl.reqs)
                else:
                    a.request_launches(ctx, d_s, d_in, d_out, wl.reqs[:50])
                    if len(wl.reqs) > 50:
                        a.batch(ctx, d_s, d_in, d_out, wl.reqs[50:])
                torch.cuda.synchronize()
                msg = first_mismatch(d_out.cpu().numpy(), want)
                assert msg is None, f"{form} at +{shift_in}, +{shift_out}: {msg}"
        plan.close()
