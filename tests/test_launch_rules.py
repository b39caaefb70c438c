"""The rules that choose a kernel for a launch (csrc/launch_rules.h), compiled
for the host alone: no GPU and no library needed."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "launch_rules.h"
using namespace aesgpu;
extern "C" int aligned(uint64_t in, uint64_t out) {
    return aligned16((const void *)in, (const void *)out);
}
extern "C" void choose(int dec, uint32_t n, const uint32_t *lengths, int ok, uint32_t n_cu,
                       uint32_t *out) {
    TileWork w;
    uint32_t max_bytes = 0;
    for (uint32_t i = 0; i < n; i++) {
        w.sum += TileWork::of(lengths[i]);
        max_bytes = lengths[i] > max_bytes ? lengths[i] : max_bytes;
    }
    const TileChoice c = choose_tiles(dec, n, max_bytes, w, ok, n_cu);
    out[0] = (uint32_t)c.kind;
    out[1] = c.nb;
    out[2] = c.parts_log2;
    out[3] = c.waves;
    out[4] = c.grid;
}
extern "C" void uneven(uint32_t n_wg, uint32_t *out) {  // [n_wg][64]
    const uint32_t inv = uneven_inverse(n_wg);
    for (uint32_t g = 0; g < n_wg; g++)
        for (uint32_t lane = 0; lane < 64; lane++)
            out[64 * g + lane] = uneven_unit(g, lane, n_wg, inv);
}
extern "C" int mixed_lanes(uint32_t n, uint32_t longest, int grouped, uint32_t n_wg,
                           uint64_t tile_bytes) {
    return mixed_chain_lanes(n, longest, (uint64_t)n * longest, grouped, n_wg, tile_bytes);
}
extern "C" int threads(uint64_t n, uint64_t units) {
    return scan_in_threads(n) + 2 * write_in_threads(n, units);
}
extern "C" int lanes(uint32_t n, uint32_t longest, uint64_t bytes, int grouped, uint32_t waves) {
    return chain_lanes_for(n, longest, bytes, grouped, waves);
}
"""
TILES, SHORT, UNEVEN = 0, 1, 2
CUS = 256


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I" + os.path.join(ROOT, "paper_1305_3345_amd", "csrc"), str(src), "-o",
                    str(so)], check=True)
    return ctypes.CDLL(str(so))


def choose(rules, lengths, dec=False, ok=True, cus=CUS):
    """(kind, blocks per lane, log2 parts, waves, workgroups) for units of these bytes."""
    out = (ctypes.c_uint32 * 5)()
    n = len(lengths)
    rules.choose(int(dec), n, (ctypes.c_uint32 * n)(*lengths), int(ok), cus, out)
    return tuple(out)


@pytest.mark.parametrize("dec", [False, True])
@pytest.mark.parametrize("lengths", [[4096], [16] * 5000, [2048] * 3000, [64, 4096] * 3000])
def test_unaligned_buffers_take_the_tile_kernels(rules, lengths, dec):
    """Only global loads may read a payload whose base is not 16-byte aligned."""
    for shift in (1, 2, 4, 8, 15):
        for a, b in ((shift, 0), (0, shift), (shift, shift)):
            ok = rules.aligned(ctypes.c_uint64(0x7F0000001000 + a),
                               ctypes.c_uint64(0x7F0000002000 + b))
            assert not ok
            assert choose(rules, lengths, dec, ok)[0] == TILES
    assert rules.aligned(ctypes.c_uint64(0x7F0000001010), ctypes.c_uint64(0x7F0000002000))


@pytest.mark.parametrize("n,longest,n_wg,mib,lanes", [
    # What was measured faster on 256 compute units (or the same: few chains).
    (8192, 64, 256, 256, 4), (8192, 512, 256, 256, 4), (8192, 2048, 256, 256, 4),
    (2048, 512, 256, 256, 4), (2048, 8192, 256, 256, 16), (8192, 64, 256, 16, 4),
    (8192, 2048, 256, 16, 16), (2048, 2048, 256, 64, 16), (8192, 512, 256, 64, 4),
    (500, 262144, 192, 90, 16),  # an uneven mix of requests: the long chains decide
    # No tiles beside the chains, and more chains than run at once.
    (48, 16, 1, 0, 16), (65, 16, 1, 0, 4), (8193, 1 << 20, 256, 16, 4)])
def test_chains_beside_tiles(rules, n, longest, n_wg, mib, lanes):
    got = rules.mixed_lanes(n, longest, 1, n_wg, ctypes.c_uint64(mib << 20))
    assert got == lanes
    assert rules.mixed_lanes(n, longest, 0, n_wg, ctypes.c_uint64(mib << 20)) == 1


@pytest.mark.parametrize("n,longest,mean,lanes", [
    (4096, 64, 64, 16), (12288, 256, 256, 16), (12288, 4096, 4096, 16),
    (12289, 256, 256, 4), (16384, 4096, 4096, 4), (16384, 1024, 1024, 4),
    (13312, 8192, 8192, 16), (16384, 65536, 65536, 16),  # long chains
    (16384, 8192, 1000, 16),  # most end early
    (16385, 16384, 16384, 4), (65536, 64, 64, 4)])  # more than run at once
def test_chains_alone(rules, n, longest, mean, lanes):
    """What was measured faster on 256 compute units of sixteen waves."""
    assert rules.lanes(n, longest, ctypes.c_uint64(n * mean), 1, 16 * CUS) == lanes
    assert rules.lanes(n, longest, ctypes.c_uint64(n * mean), 0, 16 * CUS) == 1


@pytest.mark.parametrize("lengths,dec,ctr", [
    # Nearly all of one step, parts beyond one pass: not padded to 4 KiB each.
    ([64] * 3071 + [4096], TILES, UNEVEN), ([1008] * 2499 + [4096], TILES, UNEVEN),
    ([1500] * 3071 + [4096], TILES, UNEVEN), ([64] * 2900 + [4096] * 172, TILES, UNEVEN),
    ([64] * 2480 + [4096] * 20, TILES, UNEVEN), ([64] * 2420 + [4096] * 80, SHORT, UNEVEN),
    # One pass, or enough units of two steps.
    ([64] * 2047 + [4096], SHORT, SHORT), ([64] * 2700 + [4096] * 372, SHORT, SHORT),
    ([4096] * 3072, SHORT, SHORT), ([4096] * 3073, TILES, TILES),
    # One step each.
    ([2048] * 4096, SHORT, SHORT), ([2048] * 4097, TILES, SHORT), ([1040] * 6144, TILES, SHORT),
    ([1024] * 60000, SHORT, SHORT),
    # Units over 16 KiB have sixteen parts of 2 KiB, also where few.
    ([32768], SHORT, SHORT), ([20000] * 8, SHORT, SHORT), ([32768] * 128, SHORT, SHORT),
    ([32768] * 384, SHORT, SHORT), ([32769] * 8, TILES, TILES), ([32768] * 385, TILES, TILES),
    # More than two steps take a tile kernel's single wave too long.
    ([64] * 1500 + [8192], SHORT, SHORT), ([64] * 767 + [16384], SHORT, SHORT)])
def test_short_launches_by_what_units_hold(rules, lengths, dec, ctr):
    assert choose(rules, lengths, dec=True)[0] == dec
    assert choose(rules, lengths)[0] == ctr


def dealt(rules, n_wg):
    out = np.zeros((n_wg, 64), np.uint32)
    rules.uneven(n_wg, out.ctypes.data_as(ctypes.c_void_p))
    return out


@pytest.mark.parametrize("n_wg", [1, 2, 3, 36, 37, 38, 74, 255, 256, 257, 304, 4096, 65535])
def test_uneven_units_are_dealt_once(rules, n_wg):
    """Every unit below 64 per workgroup goes to one lane of one workgroup, the
    first n units to the first lanes."""
    out = dealt(rules, n_wg)
    assert np.array_equal(np.sort(out.ravel()), np.arange(64 * n_wg))
    assert (out // n_wg == np.arange(64)).all()


@pytest.mark.parametrize("order", ["ascending", "descending", "blocks", "period"])
def test_uneven_units_in_order_of_size(rules, order):
    """The largest workgroup's parts stay near the mean for sorted lists, lists
    of blocks of one size, and flows that repeat every 512 requests (the ranges
    of consecutive units that the kernel took before hold 1.7 to 2.1 times the
    mean where a list is sorted)."""
    n = 6000
    rng = np.random.default_rng(1)
    lengths = np.exp(rng.uniform(0, np.log(4097), n)).astype(np.uint64)
    lengths = np.sort(lengths)
    if order == "descending":
        lengths = lengths[::-1]
    elif order == "blocks":
        lengths = lengths.reshape(10, -1)[rng.permutation(10)].ravel()
    elif order == "period":
        lengths = lengths[rng.integers(0, n, 512)][np.arange(n) % 512]
    parts = np.zeros(64 * CUS, np.int64)
    parts[:n] = (lengths + 1023) // 1024
    load = parts[dealt(rules, CUS)].sum(axis=1)
    # Sorted: a unit a round, and a round's units differ by one part at most.
    # Random flows: 23 or 24 units a workgroup, four standard deviations.
    limit = 1.25 if order != "period" else 1 + 4 * parts[:n].std() / parts[:n].mean() / 23 ** .5
    assert load.max() <= limit * load.mean(), (load.max(), load.mean())


@pytest.mark.parametrize("per_cu,share,kind", [
    (40, .3, UNEVEN), (40, .5, UNEVEN), (40, .7, TILES), (40, .9, TILES), (47, .6, UNEVEN), (52, .6, TILES),
    (56, .3, UNEVEN), (56, .5, TILES), (63, .3, UNEVEN), (63, .5, TILES), (63, .9, TILES)])
def test_uneven_units_that_fill_a_step(rules, per_cu, share, kind):
    """Units of 1 KiB and, by `share`, 2 KiB: the tile kernel's step."""
    n = int(per_cu * CUS / (1 + share))
    big = int(share * n)
    assert choose(rules, [2048] * big + [1024] * (n - big - 1) + [2500])[0] == kind


@pytest.mark.parametrize("per_cu", [40, 52, 63])
@pytest.mark.parametrize("lo,hi", [(1, 16001), (1, 3000)])
def test_uneven_units_of_any_size(rules, per_cu, lo, hi):
    """Log-uniform to 16 KB in tiles of 4 KiB, uniform to 3,000 B."""
    rng = np.random.default_rng(3)
    draw = rng.uniform(np.log(lo), np.log(hi), 20000) if hi > 4096 else rng.uniform(lo, hi, 20000)
    lengths = np.exp(draw) if hi > 4096 else draw
    units, parts = [], 0
    for v in lengths.astype(int):
        tiles = [4096] * (v // 4096) + ([v % 4096] if v % 4096 else [])
        units += tiles
        parts += sum((t + 1023) // 1024 for t in tiles)
        if parts >= per_cu * CUS:
            break
    assert choose(rules, units)[0] == UNEVEN


@pytest.mark.parametrize("n,tiles,use", [
    (1, 1, 0), (8191, 16, 0), (8192, 1, 0), (8192, 7, 0), (8192, 8, 2), (12000, 16, 2),
    (16383, 1, 0), (16384, 1, 3), (65536, 1, 3), (1 << 20, 16, 3)])
def test_host_threads(rules, n, tiles, use):
    """Bit 0: the scan, bit 1: writing the unit records."""
    assert rules.threads(ctypes.c_uint64(n), ctypes.c_uint64(n * tiles)) == use
