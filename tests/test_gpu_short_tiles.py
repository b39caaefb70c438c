"""GPU parity of the kernels for short launches (a unit spread over several
waves, rolled rounds) at the edges of their shapes, byte for byte against the
CPU oracle: units of a part (1 or 2 KiB) minus one block, whole, plus one
block and up to the tile size, ragged CTR tails and counters that wrap inside
a request, one pass and several, the last number of units they take and the
first they leave to the tile kernels, tiles of 4 to 16 KiB, every operation
and key size, out of place and in place; and single requests by value, CBC
decryption in place among them (one workgroup over many passes)."""
import numpy as np
import pytest
import torch

from synth import gen, workloads
from tests.gpu_util import ag, device_schedules, first_mismatch, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

OPS = {"ctr": workloads.OP_CTR, "cbc_dec": workloads.OP_CBC_DEC, "ecb_enc": 3, "ecb_dec": 4}


@pytest.fixture(scope="module")
def ctx():
    print("\n[gpu] context for short launch tests", flush=True)
    c = ag().Context(0)
    yield c
    c.close()


@pytest.fixture()
def fresh(ctx):
    cfg = ctx.get_config()
    yield ctx
    ctx.set_config(**cfg)


def requests(op, lengths, seed):
    n = len(lengths)
    reqs = np.zeros(n, workloads.REQ_DTYPE)
    reqs["length"] = np.asarray(lengths, np.uint64)
    reqs["offset"][1:] = np.cumsum((reqs["length"] + 15) // 16 * 16 + 16)[:-1]
    reqs["op"] = OPS[op]
    reqs["key_idx"] = np.arange(n) % 3
    reqs["iv"] = gen.bytes_(seed, gen.STREAM_IVS, 16 * n).reshape(n, 16)
    if op == "ctr":
        reqs["iv"][:, 8:] = 255
        reqs["iv"][:, 15] = np.arange(n) % 256  # wraps after 0 to 255 blocks
    keys, kb = workloads.make_keys(seed, 3, [128, 192, 256])
    buf = int(reqs["offset"][-1] + reqs["length"][-1] + 32)
    return workloads.Workload("short", reqs, keys, kb, buf, seed)


def sizes(op, top):
    """Lengths about the part sizes up to `top`, ragged for CTR."""
    s = sorted({v for p in (1024, 2048, 4096, 8192, 16384) for v in (p - 16, p, p + 16)
                if v <= top} | {16, 32, top})
    return s + [v - 3 for v in s] + [1, 17] if op == "ctr" else s


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("tile", [4096, 8192, 16384])
def test_unit_sizes(fresh, op, tile, inplace):
    """A few units of every size (4 or 8 waves a workgroup), and requests of
    two and three tiles."""
    print(f"[gpu] short launch: {op}, tiles of {tile}, inplace={inplace}", flush=True)
    fresh.set_config(tile_bytes=tile)
    wl = requests(op, sizes(op, 3 * tile), tile + len(op))
    inp = wl.data()
    for form in ("batch", "plan"):
        msg = first_mismatch(run_gpu(fresh, wl, inp, form=form, inplace=inplace),
                             run_oracle(wl, inp, inplace=inplace))
        assert msg is None, f"{form}: {msg}"


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", ["ctr", "cbc_dec"])
@pytest.mark.parametrize("n", [255, 257, 1024, 1025, 2049, 3072, 3073])
def test_unit_counts(fresh, op, n, inplace):
    """4 KiB units, some in requests of two: 255 and 257 (4 and 8 waves on 256
    compute units), 1,024 and 1,025 (one block per lane, two), 2,049 (a second
    pass), 3,072 and 3,073 (the last on these kernels, the first beyond)."""
    print(f"[gpu] short launch: {op}, {n} units, inplace={inplace}", flush=True)
    pairs = n // 5
    lengths = [8192] * pairs + [4096] * (n - 2 * pairs)
    np.random.default_rng(n).shuffle(lengths)
    if op == "ctr":
        lengths[0] -= 5
    wl = requests(op, lengths, n)
    inp = wl.data()
    msg = first_mismatch(run_gpu(fresh, wl, inp, form="plan", inplace=inplace),
                         run_oracle(wl, inp, inplace=inplace))
    assert msg is None, msg


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n", [4096, 4097, 20011])
def test_many_small_units(ctx, op, n, inplace):
    """Units of at most 1 KiB in any number: one pass of sixteen waves on 256
    compute units, its first unit more, and about five passes; every tail
    length of CTR."""
    print(f"[gpu] small units: {op}, {n} units, inplace={inplace}", flush=True)
    lengths = np.random.default_rng(n).integers(1, 1025, n)
    if op != "ctr":
        lengths = (lengths + 15) // 16 * 16
    wl = requests(op, lengths, n)
    inp = wl.data()
    msg = first_mismatch(run_gpu(ctx, wl, inp, form="plan", inplace=inplace),
                         run_oracle(wl, inp, inplace=inplace))
    assert msg is None, msg


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
def test_requests_by_value(ctx, op, inplace):
    """One request per launch: one block to 12 MiB and a block (the first size
    beyond these kernels where the parts spread over the device)."""
    a = ag()
    big = [65536, 262144 + 48, (12 << 20) + 16] if op in ("ctr", "cbc_dec") else [65536 + 32]
    for length in sizes(op, 16384 + 16) + big:
        print(f"[gpu] short request: {op} {length} B, inplace={inplace}", flush=True)
        wl = requests(op, [length, 16], length)
        inp = wl.data()
        d_s = device_schedules(wl)
        d_in = torch.from_numpy(inp.copy()).cuda()
        d_out = d_in if inplace else torch.from_numpy(workloads.sentinel(inp.size)).cuda()
        for r in wl.reqs:
            a.request_launch(ctx, d_s, d_in, d_out, r)
        torch.cuda.synchronize()
        msg = first_mismatch(d_out.cpu().numpy(), run_oracle(wl, inp, inplace=inplace))
        assert msg is None, f"{length}: {msg}"


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("op", list(OPS))
@pytest.mark.parametrize("n", [1, 31, 32, 33])
def test_units_among_arguments(fresh, op, n, inplace):
    """Calls of up to 32 units, whose table travels among the kernel's
    arguments, and the first beyond: whole and ragged units up to 4 KiB, and
    two calls in a row with other requests."""
    print(f"[gpu] inline units: {op}, {n} units, inplace={inplace}", flush=True)
    for seed in (n, n + 100):
        lengths = np.random.default_rng(seed).integers(1, 257, n) * 16
        if op == "ctr":
            lengths[-1] -= 7
        wl = requests(op, lengths, seed)
        inp = wl.data()
        for form in ("single", "batch"):
            msg = first_mismatch(run_gpu(fresh, wl, inp, form=form, inplace=inplace),
                                 run_oracle(wl, inp, inplace=inplace))
            assert msg is None, f"{form}: {msg}"


@pytest.mark.parametrize("op", ["ctr", "ecb_enc"])
@pytest.mark.parametrize("n,top", [(2600, 16001), (5000, 9000), (9000, 2500)])
def test_uneven_units(ctx, op, n, top):
    """Encryption-side units of uneven sizes (log-uniform lengths): a
    workgroup's units share its waves' parts, over two to four passes."""
    print(f"[gpu] uneven units: {op}, {n} requests to {top} B", flush=True)
    lengths = np.exp(np.random.default_rng(n).uniform(0, np.log(top), n)).astype(np.uint64)
    if op != "ctr":
        lengths = (lengths + np.uint64(15)) // np.uint64(16) * np.uint64(16)
    for inplace in (False, True):
        wl = requests(op, lengths, n)
        inp = wl.data()
        for form in ("plan", "batch"):
            msg = first_mismatch(run_gpu(ctx, wl, inp, form=form, inplace=inplace),
                                 run_oracle(wl, inp, inplace=inplace))
            assert msg is None, f"{form} inplace={inplace}: {msg}"
