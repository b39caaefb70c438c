"""A call whose launch is refused after its first kernel has started (in place,
the predecessor snapshots come first; one workgroup cannot hold both table sets
of a fused batch, which the launcher rejects on the host): the call reports the
error, and the calls behind it, through the same staging slots and more, give
the oracle's bytes."""
import numpy as np
import pytest
import torch

from synth import workloads
from tests.gpu_util import ag, device_schedules, first_mismatch, run_oracle
from tests.test_gpu_capture import CTR, DEC, ENC, workload

pytestmark = pytest.mark.gpu


def test_calls_after_a_refused_launch():
    print("[gpu] refused fused launch, then eight calls", flush=True)
    a = ag()
    bad = workload([ENC, DEC, CTR] * 2000, [320, 12288, 48] * 2000, seed=1)
    d_bad = torch.from_numpy(bad.data()).cuda()
    s_bad = device_schedules(bad)
    good = [workload([CTR, DEC] * 300, [160 + 16 * k, 8192] * 300, seed=k) for k in range(8)]
    bufs = [(wl, device_schedules(wl), torch.from_numpy(wl.data()).cuda(),
             torch.from_numpy(workloads.sentinel(wl.data().size)).cuda()) for wl in good]
    torch.cuda.synchronize()
    with a.Context(0) as ctx:
        cfg = ctx.get_config()
        ctx.set_config(grid=1)
        for _ in range(4):
            with pytest.raises(a.AesError) as e:
                a.batch(ctx, s_bad, d_bad, d_bad, bad.reqs)
            assert e.value.status == a.AES_ERR_DEVICE
        ctx.set_config(**cfg)
        for wl, s, d_in, d_out in bufs:
            a.batch(ctx, s, d_in, d_out, wl.reqs)
        torch.cuda.synchronize()
    assert np.array_equal(d_bad.cpu().numpy(), bad.data()), "the refused batch wrote something"
    for k, (wl, _, _, d_out) in enumerate(bufs):
        msg = first_mismatch(d_out.cpu().numpy(), run_oracle(wl, wl.data()))
        assert msg is None, f"call {k}: {msg}"
