"""Workloads for timing the library from the outside: what a program that uses
it has it do, through the Python binding's public calls, over the range of
request counts, sizes, operations, key sizes and call forms.

A case is a dict of plain values:
  form      "single" (aes_*_batch of one operation, request arrays on the
            host), "batch" / "noalloc" (request records, any operations),
            "plan" (a resident plan), "graph" (a plan captured in a HIP
            graph), "request" (one request, one launch), "serve" (the
            persistent engine, a burst of requests)
  op        "ctr", "cbc_dec", "cbc_enc", "ecb_enc", "ecb_dec", or a mix:
            "mixed" (CTR half, CBC encryption and decryption a quarter each),
            "tiles" (the four operations that run block-parallel),
            "cbc" (CBC encryption and decryption, half each)
  bits      key size, or 0 for keys of 128 and 256 bits, half each
  n         requests
  lo, hi    request bytes: log-uniform between the two, in steps of `step`
  keys      schedules, requests pick one at random
  in_place  output written over the input
  counter   "zero" or "random" low half of a CTR request's first counter block

Every output is bytes, equal or wrong: there is nothing to be near to, so no
64-bit reference is given here.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1305_3345_amd import aesgpu

OPS = {"cbc_enc": aesgpu.AES_OP_CBC_ENC, "cbc_dec": aesgpu.AES_OP_CBC_DEC,
       "ctr": aesgpu.AES_OP_CTR, "ecb_enc": aesgpu.AES_OP_ECB_ENC,
       "ecb_dec": aesgpu.AES_OP_ECB_DEC}
MIXES = {"mixed": ("ctr", "ctr", "cbc_enc", "cbc_dec"),
         "tiles": ("ctr", "cbc_dec", "ecb_enc", "ecb_dec"),
         "cbc": ("cbc_enc", "cbc_dec")}
SINGLE = {"ctr": aesgpu.ctr_batch, "cbc_dec": aesgpu.cbc_decrypt_batch,
          "cbc_enc": aesgpu.cbc_encrypt_batch, "ecb_enc": aesgpu.ecb_encrypt_batch,
          "ecb_dec": aesgpu.ecb_decrypt_batch}
PAGE = 4096
MAX_BYTES = 256 << 20  # payload of a drawn case
MAX_CHAIN = 256 << 10  # longest CBC-encrypt request of a drawn case


def _case(name, form, op, bits, n, lo, hi, step=16, keys=16, in_place=False, counter="zero"):
    return {"name": name, "form": form, "op": op, "bits": bits, "n": n, "lo": lo, "hi": hi,
            "step": step, "keys": keys, "in_place": in_place, "counter": counter}


def listed():
    return [
        # One page of an encrypted file or block device: the smallest call.
        _case("page_ctr128", "single", "ctr", 128, 1, PAGE, PAGE, keys=1),
        # A read-ahead window of 128 KiB decrypted page by page.
        _case("readahead_dec256", "single", "cbc_dec", 256, 32, PAGE, PAGE, keys=1),
        # A write-back of 256 dirty pages: CBC encryption, one key.
        _case("writeback_enc128", "single", "cbc_enc", 128, 256, PAGE, PAGE, keys=1),
        # Packets and file tails of any length, in place, counters anywhere.
        _case("ragged_ctr192", "batch", "ctr", 192, 3001, 1, 16001, step=1, keys=64,
              in_place=True, counter="random"),
        # One request launched on its own: a point of the 4 KiB .. 1 MiB sweep.
        _case("request_ecb128", "request", "ecb_enc", 128, 1, 64 << 10, 64 << 10, keys=1),
        # Extents of a file decrypted in place, the same launch again and again.
        _case("extents_dec128", "graph", "cbc_dec", 128, 192, 16 << 10, 256 << 10, step=PAGE,
              in_place=True),
        # 65,536 pages, 16 keys: the plain call, metadata handed over each time.
        _case("pages_ctr128", "single", "ctr", 128, 65536, PAGE, PAGE),
        # 65,536 pages, 16 keys: the resident plan, the other table set and key size.
        _case("pages_dec256", "plan", "cbc_dec", 256, 65536, PAGE, PAGE),
        # An uneven mix of callers: every mode in one batch, two key sizes.
        _case("mixed_2000", "batch", "mixed", 0, 2000, PAGE, 256 << 10, step=PAGE, keys=64,
              counter="random"),
        # 4,096 long serial chains.
        _case("chains_enc256", "plan", "cbc_enc", 256, 4096, 64 << 10, 64 << 10, keys=1),
        # One long stream in 16 MiB requests.
        _case("stream_ctr256", "plan", "ctr", 256, 64, 16 << 20, 16 << 20, keys=1,
              counter="random"),
        # A burst at the persistent engine: pages to 64 KiB, both CBC directions.
        _case("serve_cbc128", "serve", "cbc", 128, 64, PAGE, 64 << 10, step=PAGE),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(("single", "single", "batch", "noalloc", "plan", "graph", "request",
                       "serve"))
    if form == "serve":
        op = rng.choice(("cbc", "cbc", "tiles"))
    elif form in ("batch", "noalloc"):
        op = rng.choice(("mixed", "tiles", "ctr", "cbc_dec"))
    else:
        op = rng.choice(tuple(OPS))
    chains = op in ("cbc_enc", "mixed", "cbc")
    if form == "request":
        n, lo = 1, _log_int(rng, 16, 64 << 10 if chains else 1 << 20)
        hi = lo
    else:
        top = 64 << 10 if form == "serve" else MAX_CHAIN if chains else 4 << 20
        lo = _log_int(rng, 16, top)
        hi = lo if rng.random() < 0.5 else _log_int(rng, lo, top)
        most = 128 if form == "serve" else 16384 if chains else 65536
        n = _log_int(rng, 1, max(1, min(most, MAX_BYTES // hi)))
    step = 1 if op == "ctr" and rng.random() < 0.5 else 16
    lo = max(step, lo // step * step)
    hi = max(lo, hi // step * step)
    bits = 0 if op in MIXES and rng.random() < 0.5 else rng.choice((128, 192, 256))
    return {"form": form, "op": op, "bits": bits, "n": n, "lo": lo, "hi": hi, "step": step,
            "keys": min(n, _log_int(rng, 1, 64)), "in_place": rng.random() < 0.3,
            "counter": rng.choice(("zero", "random"))}


def _requests(case, seed):
    """The request records of a case, packed from offset 0 on 16-byte
    boundaries, and the bytes of the buffer that holds them."""
    rng = np.random.default_rng(seed)
    n, lo, hi, step = case["n"], case["lo"], case["hi"], case["step"]
    if lo == hi:
        length = np.full(n, lo, np.uint64)
    else:
        # The same sizes for every seed, in another order: the buffer keeps its size.
        length = np.exp(np.random.default_rng(n).uniform(math.log(lo), math.log(hi), n))
        length = np.clip(np.rint(length / step) * step, lo, hi).astype(np.uint64)
        rng.shuffle(length)
    reqs = np.zeros(n, aesgpu.REQ_DTYPE)
    padded = (length + np.uint64(15)) & ~np.uint64(15)
    ends = np.cumsum(padded)
    reqs["offset"] = ends - padded
    reqs["length"] = length
    reqs["key_idx"] = rng.integers(0, case["keys"], n, dtype=np.uint32)
    if case["op"] in MIXES:
        mix = np.array([OPS[o] for o in MIXES[case["op"]]], np.uint32)
        reqs["op"] = mix[rng.integers(0, mix.size, n)]
    else:
        reqs["op"] = OPS[case["op"]]
    reqs["iv"] = rng.integers(0, 256, (n, 16), dtype=np.uint8)
    if case["counter"] == "zero":
        reqs["iv"][reqs["op"] == aesgpu.AES_OP_CTR, 8:] = 0
    return reqs, int(ends[-1])


def _schedules(case, seed):
    rng = np.random.default_rng(seed + (1 << 32))
    keys = rng.integers(0, 256, (case["keys"], 32), dtype=np.uint8)
    bits = case["bits"] or np.where(rng.integers(0, 2, case["keys"]) > 0, 256, 128)
    return aesgpu.expand_keys(keys, bits)


_kept = {}  # one context and one server per process, as a program keeps them


def _context():
    if "ctx" not in _kept:
        _kept["ctx"] = aesgpu.Context(0)
    return _kept["ctx"]


SLOTS = 8192


def _server():
    """The persistent engine, and the next free of its key slots.  Its kernel
    leaves after 2 ms without requests, so that a wait for the whole device
    ends soon after the last burst."""
    if "srv" not in _kept:
        _kept["srv"] = aesgpu.Server(_context(), key_slots=SLOTS, idle_timeout_ms=2)
        _kept["slot"] = 0
    return _kept["srv"]


def prepare(case, seed):
    reqs, nbytes = _requests(case, seed)
    scheds = _schedules(case, seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    src = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=gen)
    dst = src if case["in_place"] else torch.zeros_like(src)
    s = {"form": case["form"], "op": case["op"], "reqs": reqs, "src": src, "dst": dst,
         "ctx": _context()}
    form = case["form"]
    if form == "serve":
        srv = s["srv"] = _server()
        base = _kept["slot"]
        if base + len(scheds) > SLOTS:
            base = 0
        _kept["slot"] = base + len(scheds)
        for i, k in enumerate(scheds):
            srv.set_key(base + i, k)
        reqs["key_idx"] += base
        s["posts"] = [(int(r["op"]), int(r["key_idx"]), r["iv"].copy(),
                       src.data_ptr() + int(r["offset"]), dst.data_ptr() + int(r["offset"]),
                       int(r["length"])) for r in reqs]
        torch.cuda.synchronize()  # the engine does not follow torch's stream
        return s
    s["sched"] = aesgpu.schedules_to_device(scheds)
    if form == "single":
        s["args"] = [np.ascontiguousarray(reqs[f]) for f in ("offset", "length", "key_idx", "iv")]
    elif form in ("plan", "graph"):
        s["plan"] = aesgpu.Plan(s["ctx"], reqs, len(scheds), nbytes)
        if form == "graph":
            s["graph"] = aesgpu.Graph.of_plan(s["plan"], s["sched"], src, dst)
    return s


def run(s):
    form = s["form"]
    if form == "single":
        SINGLE[s["op"]](s["ctx"], s["sched"], s["src"], s["dst"], *s["args"])
    elif form == "batch":
        aesgpu.batch(s["ctx"], s["sched"], s["src"], s["dst"], s["reqs"])
    elif form == "noalloc":
        aesgpu.batch_noalloc(s["ctx"], s["sched"], s["src"], s["dst"], s["reqs"])
    elif form == "plan":
        s["plan"].launch(s["sched"], s["src"], s["dst"])
    elif form == "graph":
        s["graph"].launch()
    elif form == "request":
        aesgpu.request_launch(s["ctx"], s["sched"], s["src"], s["dst"], s["reqs"][0])
    else:
        tickets = [s["srv"].submit(*p) for p in s["posts"]]
        status = [int(s["srv"].wait(t)["status"]) for t in tickets]
        return {"out": s["dst"], "status": np.array(status)}
    return {"out": s["dst"]}


def work(case):
    """Bytes a pass cannot do without: the payload read and written once, the
    request records and the key schedules read once.  No floating-point or
    matrix arithmetic is counted: the cipher has none."""
    reqs, _ = _requests(case, 0)
    return {"bytes": 2.0 * float(reqs["length"].sum()) + reqs.nbytes + 512.0 * case["keys"],
            "flops": 0.0}
