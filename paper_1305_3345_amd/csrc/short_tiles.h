// short_tiles.h -- the parallel modes (CTR, ECB, CBC decryption) for launches
// that are over within a few passes of the device's waves.
//
// Such a launch is bound by latencies: the unit record, the payload behind it,
// the table fill, and a wave's own way through its unit (a wave alone took
// 11,000 to 13,000 clocks for 4 KiB in the tile kernels, whose unrolled rounds
// are also several times the code to fetch).  So here: a unit is spread over
// several waves, NB blocks per lane each, so that few units occupy all compute
// units; the rounds are one loop for all key sizes, with the round keys in one
// register, a word per lane, read back with v_readlane; the fill waits for
// none of the other loads; and a pass loads the next one's payload before its
// own rounds.  One 4 KiB page takes 4.5 us (8.6 in the tile kernel), 32 pages
// of AES-256 CBC decryption 6.6 (20.1), one 64 KiB request by value 4.8 (10.6
// in the kernel with a wave per tile).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "aes_rounds.h"
#include "internal.h"

namespace aesgpu {

// 16 bytes at byte offset off of [base, base + nbytes), zeros for blocks not
// inside (nbytes a multiple of 16): a buffer load, so there is no branch.  base is
// 16-byte aligned (aligned16 in launch_rules.h).
__device__ __forceinline__ void buffer_block(const uint8_t *base, uint32_t nbytes, uint32_t off,
                                             uint32_t x[4]) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, nbytes, 0x00027000);
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
}

// The first n bytes (1..15) of a block, the rest zero: at most one load each
// of 8, 4, 2 and 1 bytes, all in flight together and none past the end (a loop
// over the bytes waited for each: 65,536 CTR units of 1 to 1,024 B took 92.7 us
// with it, 63.7 without).
__device__ __forceinline__ void load_tail(const uint8_t *p, uint32_t n, uint32_t x[4]) {
    uint2 a = make_uint2(0u, 0u);
    uint32_t b = 0u, c = 0u, d = 0u;
    if (n & 8u)
        a = *reinterpret_cast<const uint2 *>(p);
    if (n & 4u)
        b = *reinterpret_cast<const uint32_t *>(p + (n & 8u));
    if (n & 2u)
        c = *reinterpret_cast<const uint16_t *>(p + (n & 12u));
    if (n & 1u)
        d = p[n & 14u];
    const uint32_t t = c | d << ((n & 2u) << 3);  // the last one to three bytes
    const uint32_t lo = n & 4u ? b : t, hi = n & 4u ? t : 0u;
    x[0] = n & 8u ? a.x : lo;
    x[1] = n & 8u ? a.y : hi;
    x[2] = n & 8u ? lo : 0u;
    x[3] = n & 8u ? hi : 0u;
}

// Stores the first n bytes (1..15) of a block, in the same pieces.  (Chosen
// with masks: a choice between elements of o would be made between their
// addresses and put o into scratch memory.)
__device__ __forceinline__ void store_tail(uint8_t *p, uint32_t n, const uint32_t o[4]) {
    const uint32_t m8 = 0u - ((n >> 3) & 1u), m4 = 0u - ((n >> 2) & 1u);
    if (n & 8u)
        *reinterpret_cast<uint2 *>(p) = make_uint2(o[0], o[1]);
    const uint32_t lo = (o[2] & m8) | (o[0] & ~m8), hi = (o[3] & m8) | (o[1] & ~m8);
    if (n & 4u)
        *reinterpret_cast<uint32_t *>(p + (n & 8u)) = lo;
    const uint32_t t = (hi & m4) | (lo & ~m4);
    if (n & 2u)
        *reinterpret_cast<uint16_t *>(p + (n & 12u)) = (uint16_t)t;
    if (n & 1u)
        p[n & 14u] = (uint8_t)(t >> ((n & 2u) << 3));
}

// One wave's part of a unit, bytes [part * NB KiB, ...) of it (at most NB KiB).
template <bool DEC, int NB>
struct Part {
    uint64_t at;      // its place in both buffers
    uint32_t nbytes;  // 0: nothing to do
    uint32_t op;
    uint32_t kreg;         // the schedule: round key word `lane` in lanes 0..59, then
                           // the record's first four words (the round count in lane 61)
    uint32_t w[4];         // CTR: nonce words and the counter of its first block;
                           // CBC: the block before it, unless `before`
    bool before;           // CBC: the block before it is in carry
    uint32_t x[NB][4], carry[4];

    // No branches: the compiler then knows which loads are in flight.  snap:
    // the block before the unit for FLAG_PRED_IN units, or NULL to read it
    // from `in`.
    __device__ __forceinline__ void load(uint32_t lane, const Unit &un, bool valid, uint32_t part,
                                         const uint4 *snap,
                                         const aes_schedule_t *__restrict__ sched,
                                         uint32_t n_sched, const uint8_t *in) {
        const uint32_t key = un.meta & META_KEY_MASK, first = part * (64u * NB);
        const bool run = valid && (uint64_t)first * 16u < un.nbytes && key < n_sched;
        const uint32_t left = run ? un.nbytes - 16u * first : 0u;
        nbytes = left < 1024u * NB ? left : 1024u * NB;
        at = un.off + 16ull * first;
        op = unit_op(un.meta);
        const aes_schedule_t *ks = sched + (key < n_sched ? key : 0u);
        constexpr uint32_t KEY_WORD =
            (DEC ? offsetof(aes_schedule_t, dk) : offsetof(aes_schedule_t, ek)) / 4;
        static_assert(offsetof(aes_schedule_t, nr) == 4, "the round count is the second word");
        kreg = reinterpret_cast<const uint32_t *>(ks)[lane < 60u ? KEY_WORD + lane : lane - 60u];
        const uint8_t *src = in + at;
#pragma unroll
        for (int i = 0; i < NB; i++)
            buffer_block(src, nbytes & ~15u, (64u * i + lane) * 16u, x[i]);
        w[0] = un.w[0];
        w[1] = un.w[1];
        if (DEC) {
            w[2] = un.w[2];
            w[3] = un.w[3];
            before = first || (un.meta & FLAG_PRED_IN);
            buffer_block(!first && snap ? reinterpret_cast<const uint8_t *>(snap) : src - 16,
                         nbytes && before && op == AES_OP_CBC_DEC ? 16u : 0u, 0u, carry);
        } else {
            const uint64_t c = (((uint64_t)un.w[3] << 32) | un.w[2]) + first;
            w[2] = (uint32_t)c;
            w[3] = (uint32_t)(c >> 32);
        }
    }

    // Everything loaded, not only issued (before a barrier behind which other
    // waves overwrite it).
    __device__ __forceinline__ void arrived() const {
#pragma unroll
        for (int i = 0; i < NB; i++)
            asm volatile("" ::"v"(x[i][0]), "v"(x[i][1]), "v"(x[i][2]), "v"(x[i][3]));
        asm volatile("" ::"v"(carry[0]), "v"(carry[1]), "v"(carry[2]), "v"(carry[3]));
    }

    __device__ __forceinline__ uint32_t round_count() const {
        return (uint32_t)__builtin_amdgcn_readlane((int)kreg, 61);
    }

    __device__ __forceinline__ void round_key(uint32_t r, uint32_t k[4]) const {
#pragma unroll
        for (uint32_t c = 0; c < 4; c++)
            k[c] = (uint32_t)__builtin_amdgcn_readlane((int)kreg, 4u * r + c);
    }

    // The part's output blocks (a partial block of CTR: the keystream).
    __device__ __forceinline__ void rounds(const uint32_t *lds, uint32_t lane,
                                           uint32_t o[NB][4]) const {
        const uint32_t L0 = (lane & 31u) << 2, nr = round_count();
        uint32_t k[4], s[NB][4];
        round_key(0, k);
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if (!DEC && op == AES_OP_CTR) {
                const uint64_t c = (((uint64_t)w[3] << 32) | w[2]) + 64u * i + lane;
                s[i][0] = w[0] ^ k[0];
                s[i][1] = w[1] ^ k[1];
                s[i][2] = __builtin_bswap32((uint32_t)(c >> 32)) ^ k[2];
                s[i][3] = __builtin_bswap32((uint32_t)c) ^ k[3];
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++)
                    s[i][j] = x[i][j] ^ k[j];
            }
        }
#pragma unroll 1
        for (uint32_t r = 1; r < nr; r++) {
            round_key(r, k);
#pragma unroll
            for (int i = 0; i < NB; i++) {
                if (DEC)
                    dec_round(lds, s[i], k, L0);
                else
                    enc_round(lds, s[i], k, L0);
            }
        }
        round_key(nr, k);
#pragma unroll
        for (int i = 0; i < NB; i++) {
            uint32_t m[4] = {0u, 0u, 0u, 0u};  // what the last round is combined with
#pragma unroll
            for (int j = 0; j < 4; j++) {
                if (DEC && op == AES_OP_CBC_DEC)
                    m[j] = shift_up(
                        i ? (uint32_t)__builtin_amdgcn_readlane((int)x[i ? i - 1 : 0][j], 63)
                          : (before ? carry[j] : w[j]),
                        x[i][j]);
                else if (!DEC && op == AES_OP_CTR)
                    m[j] = x[i][j];
            }
            if (DEC)
                dec_last(lds, s[i], k, L0 | SI_BASE, m, o[i]);
            else
                enc_last(lds, s[i], k, L0, m, o[i]);
        }
    }

    __device__ __forceinline__ void store(uint32_t lane, uint32_t o[NB][4], const uint8_t *in,
                                          uint8_t *out) const {
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const uint32_t start = (64u * i + lane) * 16u;
            if (start + 16u <= nbytes) {
                *reinterpret_cast<uint4 *>(out + at + start) =
                    make_uint4(o[i][0], o[i][1], o[i][2], o[i][3]);
            } else if (!DEC && start < nbytes) {  // a partial block (CTR)
                uint32_t m[4];
                load_tail(in + at + start, nbytes - start, m);
#pragma unroll
                for (int j = 0; j < 4; j++)
                    m[j] ^= o[i][j];
                store_tail(out + at + start, nbytes - start, m);
            }
        }
    }
};

// The passes of a workgroup of BD threads over its parts [0, n_parts), BD / 64
// at a time; n_parts is uniform over the workgroup, cur this wave's first part,
// loaded.  in_place: a part may have to read what another part of this
// workgroup overwrites (CBC decryption): then no wave stores a pass before
// every wave has loaded the next.  record(i), load(i, record, part): see
// run_parts.
template <bool DEC, int NB, uint32_t BD, class Record, class Load>
__device__ __forceinline__ void run_passes(const uint32_t *lds, uint32_t n_parts, bool in_place,
                                           Part<DEC, NB> &cur, const Record &record,
                                           const Load &load, const uint8_t *in, uint8_t *out) {
    const uint32_t lane = threadIdx.x & 63u;
    constexpr uint32_t STEP = BD / 64u;
    uint32_t i = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + STEP;
    auto ahead = record(i);
    Part<DEC, NB> nxt;
    for (uint32_t base = 0; base < n_parts; base += STEP) {
        load(i, ahead, nxt);
        i += STEP;
        ahead = record(i);
        const uint32_t nr = cur.round_count();
        const bool run = cur.nbytes && (nr == 10u || nr == 12u || nr == 14u);
        uint32_t o[NB][4];
        if (run)
            cur.rounds(lds, lane, o);
        if (DEC && in_place) {
            nxt.arrived();
            __syncthreads();
        }
        if (run)
            cur.store(lane, o, in, out);
        cur = nxt;
    }
}

// Fills the tables and runs the parts [0, n_parts) of a workgroup (n_parts >
// 0).  record(i): part i's unit record, requested a pass before load(i, record,
// part) uses it.
template <bool DEC, int NB, uint32_t BD, class Record, class Load>
__device__ __forceinline__ void run_parts(uint32_t *lds, const TableFill<DEC, BD> &fill,
                                          uint32_t n_parts, bool in_place, const Record &record,
                                          const Load &load, const uint8_t *in, uint8_t *out) {
    const uint32_t i = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Part<DEC, NB> cur;
    load(i, record(i), cur);
    __builtin_amdgcn_sched_barrier(0);  // all loads are issued before the fill waits for its own
    fill.store(lds);
    asm volatile("" ::"v"(cur.kreg));  // loaded above, not where it is used
    if (DEC)
        cur.arrived();
    __syncthreads();
    run_passes<DEC, NB, BD>(lds, n_parts, in_place, cur, record, load, in, out);
}

}  // namespace aesgpu
