"""GPU parity on both sides of the lines that csrc/launch_rules.h draws between
the kernels, byte for byte against the CPU oracle: units nearly all of one step
with a few of two, decryption units of one step each, out of place and in
place."""
import numpy as np
import pytest

from tests.gpu_util import ag, first_mismatch, run_gpu, run_oracle
from tests.test_gpu_short_tiles import OPS, requests

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = ag().Context(0)
    yield c
    c.close()


def check(ctx, op, lengths, inplace, forms=("plan", "batch")):
    if op != "ctr":
        lengths = (np.asarray(lengths) + 15) // 16 * 16
    wl = requests(op, lengths, len(lengths))
    inp = wl.data()
    want = run_oracle(wl, inp, inplace=inplace)
    for form in forms:
        msg = first_mismatch(run_gpu(ctx, wl, inp, form=form, inplace=inplace), want)
        assert msg is None, f"{form}: {msg}"


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n,small,big,n_big", [
    (2048, 64, 4096, 1), (2049, 61, 4093, 1), (3072, 1500, 4096, 3), (3072, 64, 2500, 300),
    (3072, 64, 4096, 330), (4096, 2048, 2048, 1), (4097, 2047, 2048, 1), (6145, 1040, 2048, 9)])
def test_mostly_one_step(ctx, op, n, small, big, n_big, inplace):
    print(f"[gpu] {op}: {n} units of {small} B, {n_big} of {big} B, inplace={inplace}", flush=True)
    lengths = np.full(n, small)
    lengths[np.random.default_rng(n).permutation(n)[:n_big]] = big
    check(ctx, op, lengths, inplace)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n", [1, 8, 128, 129])
def test_few_large_units(ctx, op, n, inplace):
    """Tiles of 32 KiB: units over 16 KiB, some in requests of two tiles."""
    print(f"[gpu] {op}: {n} units to 32 KiB, inplace={inplace}", flush=True)
    cfg = ctx.get_config()
    ctx.set_config(tile_bytes=32768)
    lengths = np.random.default_rng(n).integers(16385, 32769, n)
    lengths[0] = 65536 - 48 if n > 1 else 32768
    check(ctx, op, lengths, inplace)
    ctx.set_config(**cfg)
