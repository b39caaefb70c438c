// aes_tiles_short.hip -- kernels and launchers over short_tiles.h: the units of
// a small batch, or one request passed by value.  Built with kernel arguments
// preloaded into scalar registers (a wave's first loads then have their
// addresses at once).
#include <hip/hip_runtime.h>
#include <string.h>

#include "internal.h"
#include "short_tiles.h"

namespace aesgpu {

// A unit record on its way, the same in every lane (vector loads: scalar ones
// would be waited for with the table lookups).
struct RecordLoad {
    uint4 a, b;
    uint32_t u;
    bool valid;
    __device__ __forceinline__ Unit unit() const {
        Unit un;
        un.off = (uint64_t)__builtin_amdgcn_readfirstlane(a.y) << 32 |
                 (uint32_t)__builtin_amdgcn_readfirstlane(a.x);
        un.nbytes = __builtin_amdgcn_readfirstlane(a.z);
        un.meta = __builtin_amdgcn_readfirstlane(a.w);
        un.w[0] = __builtin_amdgcn_readfirstlane(b.x);
        un.w[1] = __builtin_amdgcn_readfirstlane(b.y);
        un.w[2] = __builtin_amdgcn_readfirstlane(b.z);
        un.w[3] = __builtin_amdgcn_readfirstlane(b.w);
        return un;
    }
};

// 2^parts_log2 parts per unit; workgroup g takes the next `per` units, the first
// `more` workgroups one more, so all parts of a unit are in one pass of one
// workgroup.  (Quotient and remainder come from the host: a division here would
// be a hundred instructions of cold code.)
template <bool DEC, int NB, uint32_t BD>
__global__ __launch_bounds__(BD) void k_tiles_short(
    const Unit *__restrict__ units, uint32_t per, uint16_t more, uint16_t parts_log2,
    const uint32_t *__restrict__ timg, const aes_schedule_t *__restrict__ sched, const uint8_t *in,
    uint32_t n_sched, const uint4 *__restrict__ preds, uint8_t *out) {
    __shared__ __align__(16) uint32_t lds[DEC ? LDS_DEC_WORDS : LDS_ENC_WORDS];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t lo = blockIdx.x * per + (blockIdx.x < more ? blockIdx.x : more);
    const uint32_t hi = lo + per + (blockIdx.x < more);
    const uint32_t n_parts = (hi - lo) << parts_log2, last = hi - 1u;
    const auto record = [&](uint32_t i) {
        RecordLoad r;
        r.u = lo + (i >> parts_log2);
        r.valid = r.u < hi;
        const uint4 *p = reinterpret_cast<const uint4 *>(units + (r.valid ? r.u : last));
        // A per-lane address (of the same record) makes these vector loads.
        uint32_t zero = 0;
        asm("" : "+v"(zero));
        r.a = p[zero];
        r.b = p[1 + zero];
        return r;
    };
    const auto load = [&](uint32_t i, const RecordLoad &r, Part<DEC, NB> &p) {
        p.load(lane, r.unit(), r.valid, i & ((1u << parts_log2) - 1u),
               preds ? preds + r.u : nullptr, sched, n_sched, in);
    };
    const TableFill<DEC, BD> fill(timg);
    run_parts<DEC, NB, BD>(lds, fill, n_parts, in == out, record, load, in, out);
}

// Inclusive sum over the lanes of a wave (zero enters where a row shift or a
// broadcast has no source).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
#define AESGPU_STEP(CTRL, ROWS) \
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    AESGPU_STEP(0x111, 0xF)  // row_shr:1, 2, 4, 8
    AESGPU_STEP(0x112, 0xF)
    AESGPU_STEP(0x114, 0xF)
    AESGPU_STEP(0x118, 0xF)
    AESGPU_STEP(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
    AESGPU_STEP(0x143, 0xC)  // row_bcast:31 into rows 2 and 3
#undef AESGPU_STEP
    return v;
}

// Encryption-side units of any sizes: every workgroup takes up to 64 units, and
// its waves take their 1 KiB parts in turn, empty ones left out.  The first wave
// fetches the records for all, through LDS; each wave then holds record `lane`
// and finds a part's unit with a ballot over the running sum of the parts.
// Units of a table in device memory are dealt out one by one (uneven_unit), so
// that a list in order of size loads all workgroups alike: 4,289 requests
// log-uniform to 16 KB in ascending order, AES-128 CTR, 14.4 us against 23.1 in
// runs of consecutive units, shuffled 16.6 against 18.4.  A table that is read
// over the host link (inv_wg 0) is taken in runs, whose records come together:
// 3,001 shuffled requests 21.8 us against 29.3, ascending 25.0 against 27.4.
__global__ __launch_bounds__(1024) void k_tiles_uneven(
    const Unit *__restrict__ units, uint32_t n_units, uint32_t per, uint32_t more,
    uint32_t n_wg, uint32_t inv_wg, const uint32_t *__restrict__ timg, const aes_schedule_t *__restrict__ sched, const uint8_t *in,
    uint32_t n_sched, uint8_t *out) {
    __shared__ __align__(16) uint32_t lds[LDS_ENC_WORDS + 512u];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t g = blockIdx.x;
    const uint32_t u = inv_wg ? uneven_unit(g, lane, n_wg, inv_wg)
                              : g * per + (g < more ? g : more) + lane;
    uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
    if (wave == 0u && u < n_units && lane < per + (inv_wg ? more != 0u : g < more)) {
        const uint4 *p = reinterpret_cast<const uint4 *>(units + u);
        a = p[0];
        b = p[1];
    }
    const TableFill<false, 1024> fill(timg);
    __builtin_amdgcn_sched_barrier(0);
    fill.store(lds);
    uint4 *rec = reinterpret_cast<uint4 *>(lds + LDS_ENC_WORDS) + 2u * lane;
    if (wave == 0u) {
        rec[0] = a;
        rec[1] = b;
    }
    __syncthreads();
    a = rec[0];
    b = rec[1];
    const uint32_t end = wave_prefix_sum((a.z + 1023u) >> 10);
    const uint32_t n_parts = (uint32_t)__builtin_amdgcn_readlane((int)end, 63);
    const auto record = [](uint32_t) { return 0; };
    const auto load = [&](uint32_t i, int, Part<false, 1> &p) {
        const bool valid = i < n_parts;
        const uint32_t k = valid ? (uint32_t)__builtin_popcountll(__ballot(end <= i)) : 0u;
        const auto get = [k](uint32_t v) {
            return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k);
        };
        Unit un;
        un.off = (uint64_t)get(a.y) << 32 | get(a.x);
        un.nbytes = get(a.z);
        un.meta = get(a.w);
        un.w[0] = get(b.x);
        un.w[1] = get(b.y);
        un.w[2] = get(b.z);
        un.w[3] = get(b.w);
        const uint32_t part = valid ? i - (get(end) - ((un.nbytes + 1023u) >> 10)) : 0u;
        p.load(lane, un, valid, part, nullptr, sched, n_sched, in);
    };
    Part<false, 1> cur;
    load(wave, 0, cur);
    run_passes<false, 1, 1024>(lds, n_parts, false, cur, record, load, in, out);
}

// A unit table among the kernel arguments.
struct InlineUnits {
    Unit u[INLINE_UNITS];
};

// One pass over the n units of `table`, in workgroups of four waves (parts of
// 1 KiB, so units of up to 4 KiB, 2^parts_log2 parts each).
template <bool DEC>
__global__ __launch_bounds__(256) void k_tiles_inline(
    const uint32_t *__restrict__ timg, const aes_schedule_t *__restrict__ sched, const uint8_t *in,
    uint32_t n, uint32_t parts_log2, uint32_t n_sched, uint8_t *out, InlineUnits table) {
    __shared__ __align__(16) uint32_t lds[DEC ? LDS_DEC_WORDS : LDS_ENC_WORDS];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t i = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
    const uint32_t u = i >> parts_log2;
    const Unit un = table.u[u < n ? u : 0u];
    __builtin_amdgcn_sched_barrier(0);
    const TableFill<DEC, 256> fill(timg);
    __builtin_amdgcn_sched_barrier(0);
    const auto record = [](uint32_t) { return 0; };
    const auto load = [&](uint32_t k, int, Part<DEC, 1> &p) {
        // The only pass; there is no second one to load.
        p.load(lane, un, u < n && k < 4u, i & ((1u << parts_log2) - 1u), nullptr, sched, n_sched,
               in);
    };
    run_parts<DEC, 1, 256>(lds, fill, 1u, false, record, load, in, out);
}

// One request as one unit; workgroup g takes the next `per` parts of it, the
// first `more` workgroups one more.
template <bool DEC, int NB, uint32_t BD>
__global__ __launch_bounds__(BD) void k_request_short(
    const uint32_t *__restrict__ timg, const aes_schedule_t *__restrict__ sched, const uint8_t *in,
    uint64_t off, uint32_t nbytes, uint32_t meta, uint32_t per, uint32_t more, uint64_t w01,
    uint64_t w23, uint32_t n_sched, uint8_t *out) {
    __shared__ __align__(16) uint32_t lds[DEC ? LDS_DEC_WORDS : LDS_ENC_WORDS];
    const TableFill<DEC, BD> fill(timg);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t lo = blockIdx.x * per + (blockIdx.x < more ? blockIdx.x : more);
    const uint32_t hi = lo + per + (blockIdx.x < more);
    Unit un;
    un.off = off;
    un.nbytes = nbytes;
    un.meta = meta;
    un.w[0] = (uint32_t)w01;
    un.w[1] = (uint32_t)(w01 >> 32);
    un.w[2] = (uint32_t)w23;
    un.w[3] = (uint32_t)(w23 >> 32);
    const auto record = [](uint32_t) { return 0; };
    const auto load = [&](uint32_t i, int, Part<DEC, NB> &p) {
        p.load(lane, un, lo + i < hi, lo + i, nullptr, sched, n_sched, in);
    };
    run_parts<DEC, NB, BD>(lds, fill, hi - lo, in == out, record, load, in, out);
}

#define AESGPU_SHORT(KERNEL, K, DEC_, NB_, WAVES_)                                             \
    ((DEC_) ? ((NB_) == 2      ? (K)&KERNEL<true, 2, 1024>                                     \
               : (WAVES_) == 4 ? (K)&KERNEL<true, 1, 256>                                      \
               : (WAVES_) == 8 ? (K)&KERNEL<true, 1, 512>                                      \
                               : (K)&KERNEL<true, 1, 1024>)                                    \
            : ((NB_) == 2      ? (K)&KERNEL<false, 2, 1024>                                    \
               : (WAVES_) == 4 ? (K)&KERNEL<false, 1, 256>                                     \
               : (WAVES_) == 8 ? (K)&KERNEL<false, 1, 512>                                     \
                               : (K)&KERNEL<false, 1, 1024>))

bool launch_tiles_short(bool dec, const Unit *d_units, uint32_t n_units, uint32_t max_bytes,
                        const TileWork &work, const aes_schedule_t *d_sched, uint32_t n_sched,
                        const uint32_t *d_timg, const void *d_preds, const uint8_t *d_in,
                        uint8_t *d_out, int n_cu, void *stream, int *err) {
    const TileChoice c =
        choose_tiles(dec, n_units, max_bytes, work, aligned16(d_in, d_out), (uint32_t)n_cu);
    if (c.kind == TileKind::TILES)
        return false;
    if (c.kind == TileKind::UNEVEN) {
        hipLaunchKernelGGL(k_tiles_uneven, dim3(c.grid), dim3(64 * c.waves), 0,
                           (hipStream_t)stream, d_units, n_units, n_units / c.grid, n_units % c.grid,
                           c.grid, work.host_table ? 0u : uneven_inverse(c.grid), d_timg, d_sched,
                           d_in, n_sched, d_out);
        *err = hipGetLastError();
        return true;
    }
    using K = void (*)(const Unit *, uint32_t, uint16_t, uint16_t, const uint32_t *,
                       const aes_schedule_t *, const uint8_t *, uint32_t, const uint4 *, uint8_t *);
    const K k = AESGPU_SHORT(k_tiles_short, K, dec, c.nb, c.waves);
    hipLaunchKernelGGL(k, dim3(c.grid), dim3(64 * c.waves), 0, (hipStream_t)stream, d_units,
                       n_units / c.grid, (uint16_t)(n_units % c.grid), (uint16_t)c.parts_log2,
                       d_timg, d_sched, d_in, n_sched, (const uint4 *)d_preds, d_out);
    *err = hipGetLastError();
    return true;
}

bool launch_tiles_inline(bool dec, const Unit *units, uint32_t n_units, uint32_t max_bytes,
                         const aes_schedule_t *d_sched, uint32_t n_sched, const uint32_t *d_timg,
                         const uint8_t *d_in, uint8_t *d_out, int n_cu, void *stream, int *err) {
    uint32_t lg = 0;
    while (lg < 2 && max_bytes > 1024u << lg)
        lg++;
    const uint32_t grid = ((n_units << lg) + 3) / 4;
    if (n_units > INLINE_UNITS || max_bytes > 1024u << lg || grid > (uint32_t)n_cu ||
        !aligned16(d_in, d_out))
        return false;
    InlineUnits t;
    memcpy(t.u, units, n_units * sizeof(Unit));
    hipLaunchKernelGGL(dec ? &k_tiles_inline<true> : &k_tiles_inline<false>, dim3(grid), dim3(256),
                       0, (hipStream_t)stream, d_timg, d_sched, d_in, n_units, lg, n_sched, d_out,
                       t);
    *err = hipGetLastError();
    return true;
}

bool launch_request_short(const aes_req_t &r, const aes_schedule_t *d_sched, uint32_t n_sched,
                          const uint32_t *d_timg, const uint8_t *d_in, uint8_t *d_out, int n_cu,
                          void *stream, int *err) {
    if (r.op == AES_OP_CBC_ENC || !aligned16(d_in, d_out))
        return false;
    // Decrypted in place with CBC, all parts have to be in one workgroup.
    const uint32_t n_wg = r.op == AES_OP_CBC_DEC && d_in == d_out ? 1u : (uint32_t)n_cu;
    const int nb = r.length > 16ull * 1024u * n_wg ? 2 : 1;
    const uint64_t parts = (r.length + 1024u * nb - 1) / (1024u * nb);
    if (parts > SHORT_PARTS_PER_CU * (uint64_t)n_wg && n_wg > 1)
        return false;
    const uint32_t waves = nb == 2 ? 16u : short_waves(parts, n_wg, 1);
    uint32_t grid = (uint32_t)((parts + waves - 1) / waves);
    if (grid > n_wg)
        grid = n_wg;
    uint64_t w01 = 0, w23 = 0;
    if (r.op == AES_OP_CTR) {  // nonce, then the counter as an integer
        memcpy(&w01, r.iv, 8);
        for (int i = 8; i < 16; i++)
            w23 = (w23 << 8) | r.iv[i];
    } else if (r.op == AES_OP_CBC_DEC) {
        memcpy(&w01, r.iv, 8);
        memcpy(&w23, r.iv + 8, 8);
    }
    using K = void (*)(const uint32_t *, const aes_schedule_t *, const uint8_t *, uint64_t,
                       uint32_t, uint32_t, uint32_t, uint32_t, uint64_t, uint64_t, uint32_t,
                       uint8_t *);
    const bool dec = r.op == AES_OP_CBC_DEC || r.op == AES_OP_ECB_DEC;
    const K k = AESGPU_SHORT(k_request_short, K, dec, nb, waves);
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * waves), 0, (hipStream_t)stream, d_timg, d_sched,
                       d_in, r.offset, (uint32_t)r.length, r.key_idx | (r.op << META_OP_SHIFT),
                       (uint32_t)(parts / grid), (uint32_t)(parts % grid), w01, w23, n_sched,
                       d_out);
    *err = hipGetLastError();
    return true;
}
#undef AESGPU_SHORT

}  // namespace aesgpu
