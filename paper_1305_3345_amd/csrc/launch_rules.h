// launch_rules.h -- the rules that choose a kernel and its shape for a launch,
// from sizes and alignment alone (host code, no HIP).
#pragma once

#include <stdint.h>

namespace aesgpu {

// The kernels for short launches read the payload with buffer loads, which
// may not honour the low bits of an address; the tile kernels' global loads
// take any base.  (Request offsets are multiples of 16.)
inline bool aligned16(const void *in, const void *out) {
    return !(((uintptr_t)in | (uintptr_t)out) & 15u);
}

// Units of decryption or encryption tiles: by the tile kernels, the kernels for
// short launches, or (encryption) the kernel for uneven units.
enum class TileKind { TILES, SHORT, UNEVEN };
struct TileChoice {
    TileKind kind = TileKind::TILES;
    uint32_t nb = 0, parts_log2 = 0;  // SHORT: blocks per lane; parts of nb KiB a unit
    uint32_t waves = 0, grid = 0;     // waves of a workgroup, workgroups
};

// What units hold: parts of 1 KiB, and steps of 2 KiB (what a wave of a tile
// kernel works at once).  Counted by request, so exact for tiles of whole steps.
// (Both in one word, one addition a request: they are of disjoint ranges of a
// buffer in device memory, far below 2^32 KiB.)
struct TileWork {
    uint64_t sum = 0;         // parts, steps << 32
    bool host_table = false;  // the unit table is read over the host link
    static uint64_t of(uint64_t len) {
        return ((len + 1023) >> 10) + ((len + 2047) >> 11 << 32);
    }
    uint64_t kib() const { return (uint32_t)sum; }
    uint64_t steps() const { return sum >> 32; }
};

// Where the line lies: microseconds a launch of 4 KiB units, here and with the
// tile kernels (AES-128 CTR; CBC decryption within 1): 1 to 1,024 units 8 and 9
// to 15 (the launch call itself takes 7.5), 2,048 11.2 and 16.4, 3,000 14.1 and
// 16.9, 4,096 18.4 and 17.7, 32,768 114 and 93.  In parts of 2 KiB a compute
// unit, 4,096 such units are 32.
constexpr uint32_t SHORT_PARTS_PER_CU = 24;
// Every unit takes the parts of the largest one there, so units that are nearly
// all of one step are better off elsewhere once their parts take a second pass:
// 3,072 units, AES-256 CBC decryption, none, 1%, 6% and 10% of 4 KiB among 64 B
// 15.7 / 12.2 (tile kernel), 15.7 / 14.4, 15.7 / 15.0, 15.7 / 16.0; AES-128 12.6 /
// 10.1, 12.6 / 11.7, 12.6 / 12.2, 12.7 / 12.8; CTR 11.6 / 7.0 (uneven units), 11.6
// / 7.5, 11.6 / 8.2, 11.7 / 8.8.  2,500 units (19.5 parts a compute unit) 14.1 /
// 12.1, 14.1 / 14.3, 14.2 / 14.7; 2,000 units, one pass, 12.5 / 12.4, 12.6 / 14.2.
// Decryption units of up to 2 KiB: 4,096 11.2 / 11.0, 4,200 12.3 / 11.2, 5,000 12.8 /
// 11.8 (CTR stays: 6,144 of them 13.0 / 13.8).  Units of more than 4 KiB wait
// too long for one wave of a tile kernel.
constexpr uint32_t ONE_STEP_PER_CU = 16;
inline bool mostly_one_step(bool dec, uint64_t n_units, uint64_t parts, const TileWork &w,
                            uint64_t cus) {
    const uint64_t percent = !dec ? 110 : parts > 20 * cus ? 107 : 101;
    return 100 * w.steps() < percent * n_units;
}
// Encryption-side units of uneven sizes, by the parts of 1 KiB that they have
// (fewer than two a unit, up to this many a compute unit): lengths
// log-uniform to 16 KB, tile kernel against this one, AES-192 CTR 18.1 / 16.0
// us at 28 parts a compute unit, 23.9 / 20.6 at 42, 29.4 / 23.8 at 55; ECB 14.5
// / 13.1, 17.7 / 17.1, 23.3 / 20.3.  CBC decryption gained nothing (17.8 / 18.1,
// 22.3 / 23.3, 29.2 / 27.8), and fuller units lose (4 KiB pages 18.1 / 21.4).
// Units of mostly one step that left the kernels above: 2,500 and 3,072 of 1,500 B
// with one of 4 KiB among them 10.3 / 8.4, 10.5 / 9.3.
// Units that nearly fill one step each are what the tile kernel is best at: a
// step of such a unit costs it about 18, a step of a longer unit 25, a part here
// 13, or 11 while there are few (in these units, fitted to what follows).  Of
// units of 1 and 2 KiB, 30%, 50%, 70% and 90% of them the latter, AES-128 CTR, at
// 40 parts a compute unit 17.5 / 15.7, 15.7 / 14.9, 13.7 / 14.3, 13.3 / 13.4; at 56
// 19.6 / 18.8, 17.6 / 18.7, 16.8 / 18.2, 16.8 / 17.3; at 63 22.7 / 19.9, 19.2 / 19.9,
// 17.6 / 19.9, 17.2 / 19.7; AES-256 ECB at 56 26.0 / 23.2, 24.5 / 23.2, 22.4 / 22.6,
// 21.6 / 21.2; CTR, 60%, at 52 17.4 / 18.2.
constexpr uint32_t UNEVEN_PARTS_PER_CU = 64;
inline bool uneven_pays(uint64_t n_units, const TileWork &w, bool one_step, uint64_t cus) {
    if (n_units > 64 * cus || w.kib() > UNEVEN_PARTS_PER_CU * cus)
        return false;
    if (w.kib() <= 32 * cus)  // two passes
        return one_step || w.kib() < 2 * n_units;
    const uint64_t part = w.kib() <= 48 * cus ? 11 : 13;
    return w.kib() < 2 * n_units && part * w.kib() + 14 * n_units < 32 * w.steps();
}

// The unit that workgroup wg of n_wg (at most 65,535; inv its uneven_inverse)
// takes with lane `lane`.  Round k deals units k n_wg .. k n_wg + n_wg - 1, lane k
// of workgroup wg the one at place (wg + 37 k) mod n_wg.
// (constexpr: the kernel calls it too.)
inline uint32_t uneven_inverse(uint32_t n_wg) { return 0xFFFFFFFFu / n_wg; }
constexpr uint32_t uneven_unit(uint32_t wg, uint32_t lane, uint32_t n_wg, uint32_t inv) {
    const uint32_t at = wg + 37u * lane;  // below 2^17
    const uint32_t r = at - (uint32_t)((uint64_t)at * inv >> 32) * n_wg;  // below 2 n_wg
    return lane * n_wg + (r >= n_wg ? r - n_wg : r);
}

// Waves per workgroup: as few (4, 8 or 16) as hold the parts on n_wg
// workgroups at once, and a unit's parts.
inline uint32_t short_waves(uint64_t parts, uint32_t n_wg, uint32_t unit_parts) {
    uint32_t waves = 4;
    while (waves < 16 && (unit_parts > waves || parts > (uint64_t)waves * n_wg))
        waves *= 2;
    return waves;
}

// n_units units of at most max_bytes each on n_cu compute units.
inline TileChoice choose_tiles(bool dec, uint32_t n_units, uint32_t max_bytes,
                               const TileWork &work, bool aligned, uint32_t n_cu) {
    TileChoice c;
    if (!aligned)
        return c;
    const uint32_t cus = n_cu < 65535u ? n_cu : 65535u;
    // One block per lane for one pass (of units up to 16 KiB), else two.  Units of up to 1 KiB, which
    // fill at most half of a tile kernel's step, run here in any number, one
    // block per lane: 16,384 units of 256 B 17.4 us (AES-128 CTR) against 23.3
    // there, 65,536 units of 1 KiB 59.3 against 82.8, of 1 to 1,024 B 63.7
    // against 115.5; of 2 KiB and more the tile kernels are as fast or faster.
    uint32_t nb = 1, lg = 0;
    for (;; nb++) {
        lg = 0;
        while (lg < 5 && (uint64_t)max_bytes > ((1024ull * nb) << lg))
            lg++;
        if (nb == 2 || max_bytes <= 1024 ||
            (lg <= 4 && ((uint64_t)n_units << lg) <= 16ull * cus))
            break;
    }
    const uint64_t parts = (uint64_t)n_units << lg;
    const bool one_step = parts > (uint64_t)ONE_STEP_PER_CU * cus && nb == 2 && lg <= 1 &&
                          (dec || lg == 1) &&
                          mostly_one_step(dec, n_units, parts, work, cus);
    if (lg > 4 || one_step || (parts > SHORT_PARTS_PER_CU * cus && max_bytes > 1024)) {
        if (dec || !uneven_pays(n_units, work, one_step, cus))
            return c;
        c.kind = TileKind::UNEVEN;
        c.waves = 16;
        c.grid = n_units < cus ? n_units : cus;
        return c;
    }
    c.kind = TileKind::SHORT;
    c.nb = nb;
    c.parts_log2 = lg;
    c.waves = nb == 2 ? 16u : short_waves(parts, cus, 1u << lg);
    const uint32_t per_wg = c.waves >> lg;  // units of one pass
    c.grid = (n_units + per_wg - 1) / per_wg;
    if (c.grid > cus)
        c.grid = cus;
    return c;
}

// A single-op call over tiles shares its requests, 4,096 at a time, with a few
// host threads: where there are many to check (8,192 requests of one tile 50 us
// with the threads, 32 without, 16,384 equal), and where there are many units to
// write (16,383 requests of 16 tiles, a call among others, 721 us with them, 772
// without, while the kernels take about 700).
constexpr uint64_t THREADS_MIN_REQS = 16384, THREADS_MIN_UNITS = 65536;
inline bool scan_in_threads(uint64_t n_reqs) { return n_reqs >= THREADS_MIN_REQS; }
inline bool write_in_threads(uint64_t n_reqs, uint64_t n_units) {
    return n_reqs >= THREADS_MIN_REQS ||
           (n_reqs >= THREADS_MIN_REQS / 2 && n_units >= THREADS_MIN_UNITS);
}

// Lanes per chain of a launch over n_chain chains (the longest of `longest`
// bytes, `bytes` in all) that can put max_waves waves on the device for them: 1
// unless `grouped`; 16 while every chain then runs at once, four chains to a
// wave; else 4, as a second pass over the chains would double the time.  A chain
// on 16 lanes is 1.1 to 1.3 times as fast while a SIMD holds up to three such
// waves.  With four it is as fast only where the chains are long, or of such
// lengths that most end early (together no more than three quarters of the
// slots would hold at the longest length).  Microseconds on four and on sixteen
// lanes, 256 compute units, AES-128: 12,288 chains of 256, 1,024 and 4,096 B 13.2
// / 12.9, 36.9 / 34.2, 129 / 116; 16,384 of them 12.2 / 13.0, 36.8 / 38.8, 126 /
// 130, of 8 and 16 KiB 249 / 250 and 502 / 490 (AES-256 340 / 335, 679 / 662),
// log-uniform from 16 B to 16 KiB 466 / 377; 13,000 to 14,336 chains alike.
constexpr uint32_t LONG_CHAIN_BYTES = 8192;
inline int chain_lanes_for(uint32_t n_chain, uint32_t longest, uint64_t bytes, bool grouped,
                           uint32_t max_waves) {
    if (!grouped)
        return 1;
    if (n_chain > 4ull * max_waves)
        return 4;
    return longest >= LONG_CHAIN_BYTES || bytes <= 3ull * max_waves * longest ? 16 : 4;
}

// The same for chains (the longest of `longest` bytes) that share n_wg
// workgroups of sixteen waves with encryption tiles of tile_bytes in all; with
// tiles they get up to half of the waves, and a wave that ends its chains takes
// no tiles.  So sixteen lanes, which take four times the waves, are right only
// where the chains are what the launch waits for.  On four lanes a chain works
// at about 1/156 of the rate of a compute unit's tiles (34 MB/s against 5.3
// GB/s for AES-128; both scale with the rounds).  Microseconds on four and on
// sixteen lanes: 8,192 chains of 64, 512 and 2,048 B beside 256 MiB of CTR 197 /
// 225, 198 / 230, 201 / 241 and beside 16 MiB 17.6 / 19.3, 23.2 / 23.7, 67.5 /
// 56.3; 2,048 chains of 512 and 8,192 B beside 256 MiB 186 / 197, 272 / 210.
constexpr uint32_t CHAIN_TILE_RATE = 156;
inline int mixed_chain_lanes(uint32_t n_chain, uint32_t longest, uint64_t bytes, bool grouped,
                             uint32_t n_wg, uint64_t tile_bytes) {
    const int w = tile_bytes ? chain_lanes_for(n_chain, longest, 0, grouped, 8u * n_wg)
                             : chain_lanes_for(n_chain, longest, bytes, grouped, 16u * n_wg);
    if (w == 16 && (uint64_t)longest * n_wg * CHAIN_TILE_RATE < tile_bytes)
        return 4;
    return w;
}

}  // namespace aesgpu
