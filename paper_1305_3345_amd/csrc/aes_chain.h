// aes_chain.h -- CBC encryption (SP 800-38A 6.2) for CDNA4 (gfx950): each
// request is one serial chain, run on one lane, on four lanes (one state
// column each) or on sixteen (one state byte each), with the tables of
// aes_rounds.h.  Used by the
// chain and fused batch kernels, the per-request kernel and the persistent
// server.
#pragma once

#include <hip/hip_runtime.h>

#include "aes_rounds.h"
#include "internal.h"

namespace aesgpu {

// A 32-bit word in global memory (device memory, or host memory mapped into
// the device).
typedef __attribute__((address_space(1))) uint32_t gu32;

// ------------------------------------------------------- CBC-encrypt chains

// SP 800-38A 6.2: C_j = E(P_j ^ C_(j-1)); one chain per lane, strictly serial.
// Round keys differ between lanes, so they live in VGPRs.  Lanes of one wave
// may use different key sizes: rounds run up to MAXNR (the largest Nr in the
// wave) and a lane with fewer rounds sits out the extra ones, so mixed waves
// cost MAXNR rounds per block rather than the sum over key sizes.
template <int MAXNR>
__device__ __forceinline__ void chain_run(const uint32_t *lds, uint32_t L0,
                                          const Unit &un, const uint32_t *ek, uint32_t nr,
                                          const uint8_t *in, uint8_t *out) {
    uint32_t rk[4 * (MAXNR + 1)];
#pragma unroll
    for (int i = 0; i < MAXNR + 1; i++) {
        const uint4 v = reinterpret_cast<const uint4 *>(ek)[i];
        rk[4 * i + 0] = v.x;
        rk[4 * i + 1] = v.y;
        rk[4 * i + 2] = v.z;
        rk[4 * i + 3] = v.w;
    }
    uint32_t rkl[4];  // this lane's last-round key
#pragma unroll
    for (int w = 0; w < 4; w++)
        rkl[w] = nr == 10 ? rk[40 + w] : (nr == 12 && MAXNR >= 12 ? rk[48 + w] : rk[4 * MAXNR + w]);
    uint32_t prev[4] = {un.w[0], un.w[1], un.w[2], un.w[3]};
    const uint32_t nblk = un.nbytes >> 4;
    const uint8_t *src = in + un.off;
    uint8_t *dst = out + un.off;
    constexpr uint32_t PF = 8;  // blocks fetched together: one 128-byte line per lane
    for (uint32_t b = 0; b < nblk; b += PF) {
        uint32_t x[PF][4];
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            if (b + j < nblk) {
                const uint4 v = *reinterpret_cast<const uint4 *>(src + ((b + j) << 4));
                x[j][0] = v.x;
                x[j][1] = v.y;
                x[j][2] = v.z;
                x[j][3] = v.w;
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            if (b + j < nblk) {
                uint32_t s[4];
#pragma unroll
                for (int w = 0; w < 4; w++)
                    s[w] = x[j][w] ^ prev[w] ^ rk[w];
#pragma unroll
                for (int r = 1; r < MAXNR; r++) {
                    if (r < 10 || (uint32_t)r < nr)
                        enc_round(lds, s, rk + 4 * r, L0);
                }
                const uint32_t zero[4] = {0u, 0u, 0u, 0u};
                enc_last(lds, s, rkl, L0, zero, prev);
                *reinterpret_cast<uint4 *>(dst + ((b + j) << 4)) =
                    make_uint4(prev[0], prev[1], prev[2], prev[3]);
            }
        }
    }
}

// One chain per lane; lanes of one wave may have different keys and lengths.
// A lane whose schedule is invalid (bad index or round count) does nothing.
__device__ __forceinline__ void run_chain(const uint32_t *lds, uint32_t L0,
                                          const Unit &un, const aes_schedule_t *__restrict__ sched,
                                          uint32_t n_sched, const uint8_t *in, uint8_t *out) {
    const uint32_t key = un.meta & META_KEY_MASK;
    const aes_schedule_t *ks = sched + (key < n_sched ? key : 0u);
    const uint32_t nr = key < n_sched ? ks->nr : 0u;
    const bool ok = nr == 10 || nr == 12 || nr == 14;
    const uint64_t m12 = __ballot(ok && nr == 12);
    const uint64_t m14 = __ballot(ok && nr == 14);
    if (!ok)
        return;
    if (m14)
        chain_run<14>(lds, L0, un, ks->ek, nr, in, out);
    else if (m12)
        chain_run<12>(lds, L0, un, ks->ek, nr, in, out);
    else
        chain_run<10>(lds, L0, un, ks->ek, nr, in, out);
}

// Chains of a wave: `cl` active lanes per wave (spreading few chains over more
// waves and compute units lowers nothing but the per-CU contention; each lane
// is still one serial chain).  Wave e takes chains e*cl + lane, then strides.
__device__ __forceinline__ void chain_loop(const uint32_t *lds, uint32_t L0,
                                           uint32_t lane, uint32_t e, uint32_t n_waves,
                                           uint32_t cl, const Unit *__restrict__ chains,
                                           uint32_t n_chain,
                                           const aes_schedule_t *__restrict__ sched,
                                           uint32_t n_sched, const uint8_t *in, uint8_t *out) {
    if (lane >= cl)
        return;
    for (uint64_t c = (uint64_t)e * cl + lane; c < n_chain; c += (uint64_t)n_waves * cl) {
        const Unit un = chains[c];
        run_chain(lds, L0, un, sched, n_sched, in, out);
    }
}

// ------------------------------------------------ one chain on four lanes
//
// Lane q of a quad holds state column q and does its column's four lookups,
// so a round costs four LDS reads per lane, issued one behind the other,
// instead of sixteen.  Sixteen chains per wave: the form for batches with more
// chains than sixteen lanes each would serve (chain_lanes_for).  Round keys:
// word q of each round key in VGPRs.

// Lane q of each quad receives lane (q + K) mod 4's v.
template <int K>
__device__ __forceinline__ uint32_t quad_next(uint32_t v) {
    // quad_perm selectors [1,2,3,0], [2,3,0,1], [3,0,1,2]
    constexpr int sel = K == 1 ? 0x39 : (K == 2 ? 0x4E : 0x93);
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, sel, 0xF, 0xF, false);
}

// A round of the quad form.  Column j of the round's output takes row r from
// column j + r (ShiftRows), so lane j needs Te_r of byte r of lane (j + r)'s
// column.  Each lane looks up the four bytes of its own column and the quad
// exchanges the looked-up words afterwards: the exchange then reads values
// returned by LDS, not ones a VALU op has just written, and the lookups do not
// wait for it.
// The lookup that needs no exchange goes last: the three exchanged words are
// moved while it is in flight, so only one XOR3 stands between the last LDS
// return and the next round's addresses.
__device__ __forceinline__ uint32_t quad_round_col(const uint32_t *lds, uint32_t st, uint32_t k,
                                                   uint32_t L0) {
    const uint32_t a1 = tlook<1, 1>(lds, st, L0);
    const uint32_t a2 = tlook<2, 2>(lds, st, L0);
    const uint32_t a3 = tlook<3, 3>(lds, st, L0);
    const uint32_t a0 = tlook<0, 0>(lds, st, L0);
    return xor3(xor3(quad_next<1>(a1), quad_next<2>(a2), k), quad_next<3>(a3), a0);
}

// The last round's SubBytes/ShiftRows column in the quad form (byte r of
// column j is S of byte r of lane (j + r)'s column), exchanged after lookup.
__device__ __forceinline__ uint32_t quad_sub_col(const uint32_t *lds, uint32_t st, uint32_t L0) {
    const uint32_t b = quad_next<1>(tlook<1, 0>(lds, st, L0));
    const uint32_t c = quad_next<2>(tlook<2, 1>(lds, st, L0));
    const uint32_t d = quad_next<3>(tlook<3, 2>(lds, st, L0));
    const uint32_t a = tlook<0, 3>(lds, st, L0);  // unexchanged, last
    return pick_diag(a, b, c, d);
}

// One block of a quad's chain: the whitened state st through rounds 1 ..
// MAXNR-1 and the last round.  A quad whose schedule has fewer rounds than
// MAXNR (quads of one wave may mix key sizes) runs the extra rounds too and
// takes the state it had before them into its last round: a select instead of
// a branch around each extra round, which costs two exec-mask updates and two
// taken branches per round.  With nr == MAXNR known at compile time the
// selects fold away.
template <int MAXNR>
__device__ __forceinline__ uint32_t quad_block(const uint32_t *lds, uint32_t st, const uint32_t *rk,
                                               uint32_t rkl, uint32_t nr, uint32_t L0) {
    uint32_t s10 = 0, s12 = 0;  // the state entering round 10 / round 12
#pragma unroll
    for (int r = 1; r < MAXNR; r++) {
        if (r == 10)
            s10 = st;
        if (r == 12)
            s12 = st;
        st = quad_round_col(lds, st, rk[r], L0);
    }
    if (MAXNR > 10)
        st = nr == 10u ? s10 : (MAXNR > 12 && nr == 12u ? s12 : st);
    return quad_sub_col(lds, st, L0) ^ rkl;
}

// Runs a quad's chain.  Lanes of a quad share one chain (un, ek, nr); quads
// of a wave may have different chains, keys and key sizes: rounds run up to
// MAXNR.
template <int MAXNR>
__device__ __forceinline__ void chain_quad_run(const uint32_t *lds, uint32_t L0, uint32_t q,
                                               const Unit &un, const uint32_t *ek, uint32_t nr,
                                               const uint8_t *in, uint8_t *out) {
    uint32_t rk[MAXNR + 1];
#pragma unroll
    for (int r = 0; r <= MAXNR; r++)
        rk[r] = ek[4 * r + q];
    const uint32_t rkl = nr == 10 ? rk[10] : (nr == 12 && MAXNR >= 12 ? rk[12] : rk[MAXNR]);
    // the IV's word q, selected with masks (an indexed read of un.w would
    // put the record in scratch memory)
    uint32_t prev = 0;
#pragma unroll
    for (uint32_t w = 0; w < 4; w++)
        prev |= un.w[w] & (0u - (uint32_t)(q == w));
    const uint32_t nblk = un.nbytes >> 4;
    if (nblk == 0)
        return;
    // Through the global address space: a payload pointer that the compiler
    // cannot trace to a kernel argument (the serving kernel reads it from a
    // queue unit) would otherwise be accessed with flat instructions, which
    // it also counts as LDS operations, and every round's LDS wait would then
    // be for all four lookups instead of the next one.
    const gu32 *src = (const gu32 *)(in + un.off) + q;
    gu32 *dst = (gu32 *)(out + un.off) + q;
    // Blocks go in groups of PF, software-pipelined: group g's words are
    // loaded while group g-1's rounds run, and group g-1's ciphertext is
    // stored while group g's run, so no wait falls on a load or store issued
    // less than a group earlier (waiting on the loads of the group about to
    // run cost about a seventh of a chain's time).  Loads past the chain's
    // end read its last block again (always in bounds, and no branch); the
    // whole groups run without per-block checks, a partial last group after
    // them.
    constexpr uint32_t PF = 8;
    const uint32_t last = nblk - 1u;
    const uint32_t nfull = nblk / PF * PF;
    uint32_t x[PF], y[PF];
#pragma unroll
    for (uint32_t j = 0; j < PF; j++)
        x[j] = src[4 * (j < last ? j : last)];
    uint32_t b = 0;
    for (; b < nfull; b += PF) {
        // Using the group's first word here (an empty asm with a memory
        // clobber keeps it in place) puts the wait for the group's loads
        // before the stores and loads issued below.
        uint32_t st = x[0] ^ prev ^ rk[0];
        asm volatile("" ::"v"(st) : "memory");
        if (b) {
            gu32 *d = dst + 4 * (b - PF);
#pragma unroll
            for (uint32_t j = 0; j < PF; j++)
                d[4 * j] = y[j];
        }
        uint32_t xn[PF];
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            const uint32_t i = b + PF + j;
            xn[j] = src[4 * (i < last ? i : last)];
        }
        // Keeps the loads here, a group ahead of their use (without it the
        // scheduler sinks them to the end of the group, next to the copies
        // into x, and the group ends waiting on them).
        asm volatile("" ::: "memory");
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            if (j)
                st = x[j] ^ prev ^ rk[0];
            prev = quad_block<MAXNR>(lds, st, rk, rkl, nr, L0);
            y[j] = prev;
        }
#pragma unroll
        for (uint32_t j = 0; j < PF; j++)
            x[j] = xn[j];
    }
    if (nfull) {
        gu32 *d = dst + 4 * (nfull - PF);
#pragma unroll
        for (uint32_t j = 0; j < PF; j++)
            d[4 * j] = y[j];
    }
    if (nfull < nblk) {
        gu32 *d = dst + 4 * nfull;
#pragma unroll
        for (uint32_t j = 0; j < PF - 1; j++) {
            if (nfull + j < nblk) {
                prev = quad_block<MAXNR>(lds, x[j] ^ prev ^ rk[0], rk, rkl, nr, L0);
                d[4 * j] = prev;
            }
        }
    }
}

// --------------------------------------------- one chain on sixteen lanes
//
// The shortest round: one lookup per lane.  Lane 4 b + p of a row of sixteen
// ("bank" b, place p) looks up one state byte, so a round is one LDS round
// trip, four XORs and one address op, against four lookups issued one behind
// the other in the four-lane form.  The four words of an output column are
// summed with DPP XORs of the looked-up words.  No round moves the state: two
// layouts alternate, and which byte of its word a lane looks up does the
// ShiftRows.  With column c taking row r from column c + r:
//   banks:  lane (b, p) holds column b and looks up row b - p, a part of
//           column p; summed over the four banks (row_ror), every lane of
//           place p holds column p;
//   places: lane (b, p) holds column p and looks up row p - b, a part of
//           column b; summed inside the quad, every lane of bank b holds
//           column b.
// Odd rounds go from banks to places, even rounds back.  Round 1 takes row b
// of column p + b (also a part of column p), and the last round, which has no
// sum, row b of column p: its byte lands in column p - b.  Between two blocks
// a byte therefore moves only in banks 1 and 3, by two places.  Round counts
// are even, so every block starts and ends alike.
//
// Bound by the dependent chain: clocks per round on gfx950, rounds alone, one
// wave per compute unit: 80 here (60 to 64 of them the address op, the lookup
// and its wait, 16 the four XORs) against 98 in the four-lane form.  One 16 KiB
// chain takes 365 us in place of 470 (AES-128), 508 in place of 638 (AES-256);
// 4,096 chains of 64 KiB AES-256 run at 127 GB/s in place of 102.

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// w and its three DPP moves, summed with k.  Every DPP operand is the looked-up
// word or a key, none a value that a VALU op has just written (which would need
// two wait states): two XORs with a DPP operand, one move, one three-input XOR.
template <int C1, int C2, int C3>
__device__ __forceinline__ uint32_t dpp_sum(uint32_t w, uint32_t k) {
    return xor3(k ^ dpp_mov<C1>(w), w ^ dpp_mov<C2>(w), dpp_mov<C3>(w));
}

// The word looked up at addr, summed over the four banks of a row (places
// keep theirs) or over the four places of a quad (banks keep theirs), plus k.
template <bool BANKS>
__device__ __forceinline__ uint32_t look_sum(const uint32_t *lds, uint32_t addr, uint32_t k) {
    const uint32_t w = lds_word(lds, addr);
    // The compiler keeps two instructions between a load into a register and
    // a DPP read of it and counts the wait as one: this one (the priority
    // waves have anyway) issues while the lookup is in flight, where a nop
    // would come after the wait.
    __builtin_amdgcn_s_setprio(0);
    return BANKS ? dpp_sum<0x124, 0x128, 0x12C>(w, k)  // row_ror:4, 8, 12
                 : dpp_sum<0x39, 0x4E, 0x93>(w, k);    // quad_perm rotations
}

// What a lane looks up: its table (bank slot, parity, region) and the v_perm
// selector that puts byte `row` of the state word into the address.
struct RowLook {
    uint32_t base, sel;
    __device__ __forceinline__ RowLook(uint32_t L0, uint32_t table, uint32_t row)
        : base(L0 | (table & 1u) << 7 | (table >> 1) << 16), sel(0x0C020400u | row << 8) {}
    __device__ __forceinline__ uint32_t addr(uint32_t st) const {
        return __builtin_amdgcn_perm(st, base, sel);
    }
};

// Runs the chain of a row of sixteen lanes.  Lanes of a row share one chain
// (un, ek, nr); rows of a wave may have different chains, keys and key sizes:
// rounds run up to MAXNR, as in the four-lane form.
template <int MAXNR>
__device__ __forceinline__ void chain_row_run(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                              const Unit &un, const uint32_t *ek, uint32_t nr,
                                              const uint8_t *in, uint8_t *out) {
    const uint32_t b = (lane >> 2) & 3u, p = lane & 3u;
    const RowLook to_places(L0, (b - p) & 3u, (b - p) & 3u);
    const RowLook to_banks(L0, (p - b) & 3u, (p - b) & 3u);
    const RowLook to_bytes(L0, 0u, b);  // Te0 holds S(x) in bits 8..23
    uint32_t rk[MAXNR];
#pragma unroll
    for (int r = 1; r < MAXNR; r++)
        rk[r] = ek[4 * r + (r & 1 ? p : b)];
    // Byte b of a word, at the address position (bits 8..15).
    const auto at8 = [b](uint32_t w) { return ((w >> (8u * b)) & 0xFFu) << 8; };
    // Columns of this lane's bytes, in and out.
    const uint32_t ci = (p + b) & 3u, co = (p - b) & 3u;
    const uint32_t rko = at8(ek[4 * nr + co]);
    const uint32_t rki = at8(ek[4 * nr + ci]);
    // Round 1's lookup: byte b of column ci through table b.
    const uint32_t k0 = at8(ek[ci]) ^ rki ^ RowLook(L0, b, 0).base;
    uint32_t iv = 0;
#pragma unroll
    for (uint32_t w = 0; w < 4; w++)
        iv |= un.w[w] & (0u - (uint32_t)(ci == w));
    // The last round's word of the block before: its byte of SubBytes in bits
    // 8..15, which the next block takes from this lane or, in banks 1 and 3,
    // from two places on.
    uint32_t prev = 0;
    const uint32_t own = b & 1u ? 0u : 0xFF00u, moved = own ^ 0xFF00u;
    uint32_t first = at8(iv) ^ rki;  // stands in for it before the first block
    const uint32_t nblk = un.nbytes >> 4;
    if (nblk == 0)
        return;
    typedef __attribute__((address_space(1))) uint8_t gu8;
    const gu8 *src = (const gu8 *)(in + un.off) + 4u * ci + b;
    gu8 *dst = (gu8 *)(out + un.off) + 4u * co + b;
    // One block: x is this lane's input byte as a round-1 address (whitened);
    // returns the last round's word, its byte of SubBytes in bits 8..15.
    const auto block = [&](uint32_t x) -> uint32_t {
        const uint32_t a = (dpp_mov<0x4E>(prev) & moved) ^ ((prev & own) ^ x);
        uint32_t st = look_sum<true>(lds, a, rk[1]);
        uint32_t s10 = 0, s12 = 0;  // the state entering round 10 / round 12
#pragma unroll
        for (int r = 2; r < MAXNR; r++) {
            if (r == 10)
                s10 = st;
            if (r == 12)
                s12 = st;
            st = r & 1 ? look_sum<true>(lds, to_places.addr(st), rk[r])
                       : look_sum<false>(lds, to_banks.addr(st), rk[r]);
        }
        if (MAXNR > 10)
            st = nr == 10u ? s10 : (MAXNR > 12 && nr == 12u ? s12 : st);
        prev = lds_word(lds, to_bytes.addr(st));
        return prev;
    };
    // Loads a group of blocks ahead, stores a group behind, as in the
    // four-lane form.
    constexpr uint32_t PF = 8;
    const uint32_t last = nblk - 1u;
    const uint32_t nfull = nblk / PF * PF;
    uint32_t x[PF], y[PF];
#pragma unroll
    for (uint32_t j = 0; j < PF; j++)
        x[j] = src[16 * (j < last ? j : last)];
    uint32_t blk = 0;
    for (; blk < nfull; blk += PF) {
        uint32_t a[PF];
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            a[j] = x[j] << 8 ^ (k0 ^ (j ? 0u : first));
            asm volatile("" : "+v"(a[j])::"memory");
        }
        first = 0;
        if (blk) {
            gu8 *d = dst + 16 * (blk - PF);
#pragma unroll
            for (uint32_t j = 0; j < PF; j++)
                d[16 * j] = (uint8_t)(y[j] >> 8);
        }
#pragma unroll
        for (uint32_t j = 0; j < PF; j++) {
            const uint32_t i = blk + PF + j;
            x[j] = src[16 * (i < last ? i : last)];
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (uint32_t j = 0; j < PF; j++)
            y[j] = block(a[j]) ^ rko;
    }
    if (nfull) {
        gu8 *d = dst + 16 * (nfull - PF);
#pragma unroll
        for (uint32_t j = 0; j < PF; j++)
            d[16 * j] = (uint8_t)(y[j] >> 8);
    }
    if (nfull < nblk) {
        gu8 *d = dst + 16 * nfull;
#pragma unroll
        for (uint32_t j = 0; j < PF - 1; j++) {
            if (nfull + j < nblk)
                d[16 * j] = (uint8_t)((block(x[j] << 8 ^ (k0 ^ (j ? 0u : first))) ^ rko) >> 8);
        }
    }
}

// A chain on W = 4 or 16 lanes of the calling wave; lanes of a group of W
// share un, ek and nr.
template <int W, int MAXNR>
__device__ __forceinline__ void chain_group_run(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                                const Unit &un, const uint32_t *ek, uint32_t nr,
                                                const uint8_t *in, uint8_t *out) {
    if (W == 4)
        chain_quad_run<MAXNR>(lds, L0, lane & 3u, un, ek, nr, in, out);
    else
        chain_row_run<MAXNR>(lds, L0, lane, un, ek, nr, in, out);
}

// Key check and round-count dispatch for the chains of a wave's groups of W
// lanes (un, per group); MAXNR is the largest round count among them.
template <int W>
__device__ __forceinline__ void run_chains(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                           bool active, const Unit &un,
                                           const aes_schedule_t *__restrict__ sched,
                                           uint32_t n_sched, const uint8_t *in, uint8_t *out) {
    const uint32_t key = un.meta & META_KEY_MASK;
    const bool keyed = active && key < n_sched;
    const aes_schedule_t *ks = sched + (keyed ? key : 0u);
    const uint32_t nr = keyed ? ks->nr : 0u;
    const bool ok = nr == 10 || nr == 12 || nr == 14;
    const uint64_t m12 = __ballot(ok && nr == 12);
    const uint64_t m14 = __ballot(ok && nr == 14);
    const uint64_t mok = __ballot(ok);
    if (!ok)
        return;
    // A wave whose chains all have the largest round count runs it as a
    // constant (no selects before the last round).
    if (m14 == mok)
        chain_group_run<W, 14>(lds, L0, lane, un, ks->ek, 14u, in, out);
    else if (m14)
        chain_group_run<W, 14>(lds, L0, lane, un, ks->ek, nr, in, out);
    else if (m12 == mok)
        chain_group_run<W, 12>(lds, L0, lane, un, ks->ek, 12u, in, out);
    else if (m12)
        chain_group_run<W, 12>(lds, L0, lane, un, ks->ek, nr, in, out);
    else
        chain_group_run<W, 10>(lds, L0, lane, un, ks->ek, nr, in, out);
}

// Runs one CBC-encrypt chain on the first sixteen lanes of the calling wave
// (the other lanes take no part).  Schedule and round count (10, 12 or 14) are
// wave-uniform.
__device__ __forceinline__ void run_chain_row(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                              const Unit &un, const uint32_t *ek, uint32_t nr,
                                              const uint8_t *in, uint8_t *out) {
    if (lane >= 16u)
        return;
    if (nr == 10)
        chain_row_run<10>(lds, L0, lane, un, ek, 10u, in, out);
    else if (nr == 12)
        chain_row_run<12>(lds, L0, lane, un, ek, 12u, in, out);
    else if (nr == 14)
        chain_row_run<14>(lds, L0, lane, un, ek, 14u, in, out);
}

// Chains of a wave in groups of W lanes, 64 / W chains per wave.  Wave e takes
// chains (64 / W) e + lane / W, then strides by (64 / W) n_waves.
template <int W>
__device__ __forceinline__ void chain_loop_group(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                                 uint32_t e, uint32_t n_waves,
                                                 const Unit *__restrict__ chains,
                                                 uint32_t n_chain,
                                                 const aes_schedule_t *__restrict__ sched,
                                                 uint32_t n_sched, const uint8_t *in,
                                                 uint8_t *out) {
    constexpr uint32_t PER = 64 / W;
    for (uint64_t base = (uint64_t)e * PER; base < n_chain; base += (uint64_t)n_waves * PER) {
        const uint64_t c = base + lane / W;
        const bool active = c < n_chain;
        Unit un;
        if (active) {
            un = chains[c];
        } else {
            un.off = 0;
            un.nbytes = 0;
            un.meta = 0;
            un.w[0] = un.w[1] = un.w[2] = un.w[3] = 0u;
        }
        run_chains<W>(lds, L0, lane, active, un, sched, n_sched, in, out);
    }
}

// The chains of a wave, W lanes each (W = 1: cl chains per wave).
template <int W>
__device__ __forceinline__ void chain_loop_any(const uint32_t *lds, uint32_t L0, uint32_t lane,
                                               uint32_t e, uint32_t n_waves, uint32_t cl,
                                               const Unit *__restrict__ chains, uint32_t n_chain,
                                               const aes_schedule_t *__restrict__ sched,
                                               uint32_t n_sched, const uint8_t *in,
                                               uint8_t *out) {
    if (W == 1)
        chain_loop(lds, L0, lane, e, n_waves, cl, chains, n_chain, sched, n_sched, in, out);
    else
        chain_loop_group<W>(lds, L0, lane, e, n_waves, chains, n_chain, sched, n_sched, in, out);
}

}  // namespace aesgpu
