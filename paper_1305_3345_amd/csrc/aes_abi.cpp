// aes_abi.cpp -- the C ABI: validation, planning, contexts, plans, launches.
//
// A call follows the service-request path of the paper (section 3.2): the
// caller hands over input and output buffers and a request list; the library
// checks every request on the host, cuts the requests into work units
// (section 2: one launch carries one large task or many small tasks), hands the
// unit table over (among the kernel arguments, in pinned staging that the
// kernels read, or uploaded) and launches the round kernels on the caller's
// stream.
#include <hip/hip_runtime.h>
#include <sched.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "host_pool.h"
#include "internal.h"
#include "tune_cache.h"

using namespace aesgpu;

namespace {

thread_local int g_last_hip = 0;

int hip_fail(hipError_t e) {
    g_last_hip = (int)e;
    return AES_ERR_DEVICE;
}

}  // namespace

int aesgpu::hip_fail_status(int hip_error) { return hip_fail((hipError_t)hip_error); }

namespace {

#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return hip_fail(e_);                                                                   \
    } while (0)

constexpr uint64_t MAX_REQ_BYTES = (1ull << 32) - 16;
constexpr uint32_t DEFAULT_TILE = 4096;

// ------------------------------------------------------------- validation

// The rules one request must meet (op already known to be valid), in the
// order whose first failure a call reports.
inline int check_request(uint32_t op, uint64_t off, uint64_t len, uint32_t key,
                         uint32_t n_scheds, uint64_t buf_bytes) {
    if (len > MAX_REQ_BYTES || (op != AES_OP_CTR && (len & 15)))
        return AES_ERR_LENGTH;
    if ((off & 15) || off > buf_bytes || len > buf_bytes - off || key >= n_scheds ||
        key >= MAX_KEYS)
        return AES_ERR_RANGE;
    return AES_OK;
}

// Checks one request list against buffer size and schedule count, and that
// the written byte ranges are pairwise disjoint.
int validate(const aes_req_t *reqs, uint64_t n, uint32_t n_scheds, uint64_t buf_bytes) {
    if (n && !reqs)
        return AES_ERR_ARG;
    bool sorted = true;
    uint64_t last_off = 0;
    for (uint64_t i = 0; i < n; i++) {
        const aes_req_t &r = reqs[i];
        if (r.op > AES_OP_ECB_DEC)
            return AES_ERR_ARG;
        const int st = check_request(r.op, r.offset, r.length, r.key_idx, n_scheds, buf_bytes);
        if (st)
            return st;
        if (r.length) {
            if (r.offset < last_off)
                sorted = false;
            last_off = r.offset;
        }
    }
    // Disjointness: a linear scan when the requests come in offset order
    // (the common case), else a sort of (offset, end) pairs.
    if (sorted) {
        uint64_t end = 0;
        bool any = false;
        for (uint64_t i = 0; i < n; i++) {
            if (!reqs[i].length)
                continue;
            if (any && reqs[i].offset < end)
                return AES_ERR_OVERLAP;
            end = reqs[i].offset + reqs[i].length;
            any = true;
        }
        return AES_OK;
    }
    std::vector<std::pair<uint64_t, uint64_t>> ranges;
    try {
        ranges.reserve(n);
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    for (uint64_t i = 0; i < n; i++)
        if (reqs[i].length)
            ranges.emplace_back(reqs[i].offset, reqs[i].offset + reqs[i].length);
    std::sort(ranges.begin(), ranges.end());
    for (size_t i = 1; i < ranges.size(); i++)
        if (ranges[i].first < ranges[i - 1].second)
            return AES_ERR_OVERLAP;
    return AES_OK;
}

bool is_dec_tile_op(uint32_t op) { return op == AES_OP_CBC_DEC || op == AES_OP_ECB_DEC; }
bool is_enc_tile_op(uint32_t op) { return op == AES_OP_CTR || op == AES_OP_ECB_ENC; }

// What one pass over a request list finds: tiles (for CBC encryption: chains)
// and bytes by operation, and whether the nonempty requests come in offset
// order without overlapping (if not, check_disjoint decides).
struct BatchScan {
    uint64_t units[5] = {0, 0, 0, 0, 0}, bytes[5] = {0, 0, 0, 0, 0};
    uint64_t work[5] = {0, 0, 0, 0, 0};  // sums of TileWork::of
    uint64_t longest = 0;  // bytes of the longest request with tiles
    uint64_t longest_chain = 0;
    bool ordered = true, pred_in = false;
    uint64_t n_dec() const { return units[AES_OP_CBC_DEC] + units[AES_OP_ECB_DEC]; }
    uint64_t n_enc() const { return units[AES_OP_CTR] + units[AES_OP_ECB_ENC]; }
    uint64_t n_chain() const { return units[AES_OP_CBC_ENC]; }
    uint64_t n_units() const { return n_dec() + n_enc() + n_chain(); }
    uint64_t dec_bytes() const { return bytes[AES_OP_CBC_DEC] + bytes[AES_OP_ECB_DEC]; }
    uint64_t enc_bytes() const { return bytes[AES_OP_CTR] + bytes[AES_OP_ECB_ENC]; }
    TileWork dec_work() const { return {work[AES_OP_CBC_DEC] + work[AES_OP_ECB_DEC]}; }
    TileWork enc_work() const { return {work[AES_OP_CTR] + work[AES_OP_ECB_ENC]}; }
};

inline uint64_t tile_count(uint64_t len, uint32_t tile) {
    return len <= tile ? 1 : (len + tile - 1) / tile;  // most requests: no division
}

// The per-request rules of validate, in its order of errors.
int scan_requests(const aes_req_t *reqs, uint64_t n, uint32_t n_scheds, uint64_t buf_bytes,
                  uint32_t tile, BatchScan &b) {
    uint64_t end = 0, longest = 0, longest_chain = 0;
    bool ordered = true, pred_in = false;
    for (uint64_t i = 0; i < n; i++) {
        const aes_req_t &r = reqs[i];
        if (r.op > AES_OP_ECB_DEC)
            return AES_ERR_ARG;
        const int st = check_request(r.op, r.offset, r.length, r.key_idx, n_scheds, buf_bytes);
        if (st)
            return st;
        if (!r.length)
            continue;
        ordered &= r.offset >= end;
        end = r.offset + r.length;
        b.bytes[r.op] += r.length;
        b.work[r.op] += TileWork::of(r.length);
        if (r.op == AES_OP_CBC_ENC) {
            b.units[r.op]++;
            longest_chain = std::max(longest_chain, r.length);
            continue;
        }
        longest = std::max(longest, r.length);
        const uint64_t t = tile_count(r.length, tile);
        b.units[r.op] += t;
        pred_in |= r.op == AES_OP_CBC_DEC && t > 1;
    }
    b.longest = longest;
    b.longest_chain = longest_chain;
    b.ordered = ordered;
    b.pred_in = pred_in;
    return AES_OK;
}

// The disjointness rule for a list that is not in order; ranges has
// room for every nonempty request.
int check_disjoint(const aes_req_t *reqs, uint64_t n, std::pair<uint64_t, uint64_t> *ranges) {
    uint64_t k = 0;
    for (uint64_t i = 0; i < n; i++)
        if (reqs[i].length)
            ranges[k++] = {reqs[i].offset, reqs[i].offset + reqs[i].length};
    std::sort(ranges, ranges + k);
    for (uint64_t i = 1; i < k; i++)
        if (ranges[i].first < ranges[i - 1].second)
            return AES_ERR_OVERLAP;
    return AES_OK;
}

int check_buffers(const uint8_t *d_in, const uint8_t *d_out, uint64_t buf_bytes, uint64_t n,
                  const void *d_scheds) {
    if (!n)
        return AES_OK;
    if (!d_in || !d_out || !d_scheds)
        return AES_ERR_ARG;
    if (d_in != d_out) {
        const uintptr_t a = (uintptr_t)d_in, b = (uintptr_t)d_out;
        if (a < b + buf_bytes && b < a + buf_bytes)
            return AES_ERR_OVERLAP;
    }
    return AES_OK;
}

// ---------------------------------------------------------------- planner

inline uint32_t le32(const uint8_t *p) {
    uint32_t v;
    memcpy(&v, p, 4);
    return v;
}

inline uint64_t be64(const uint8_t *p) {
    uint64_t v;
    memcpy(&v, p, 8);
    return __builtin_bswap64(v);
}

struct Planned {
    std::vector<Unit> dec;     // CBC- and ECB-decrypt tiles
    std::vector<Unit> ctr;     // CTR tiles, then ECB-encrypt tiles (the last n_ecb)
    std::vector<Unit> chains;  // CBC-encrypt chains, longest first, ties by key
    uint64_t payload = 0;
    uint64_t extent = 0;
    uint64_t dec_bytes = 0, ctr_bytes = 0, chain_bytes = 0;
    uint32_t max_tile = 0;  // bytes of the largest tile
    TileWork dec_work, enc_work;
    bool dec_has_pred_in = false;
    size_t n_ecb = 0;  // ECB-encrypt tiles at the end of ctr
    std::vector<Unit> ecb;       // ECB-encrypt tiles while planning (appended to ctr)
    std::vector<Unit> sort_buf;  // scratch of the key grouping

    // Empties the plan and keeps the vectors' storage: a context reuses one
    // Planned for every single-call batch, so a call touches no fresh pages.
    void reset() {
        dec.clear();
        ctr.clear();
        ecb.clear();
        chains.clear();
        payload = extent = 0;
        max_tile = 0;
        dec_work = enc_work = TileWork();
        dec_bytes = ctr_bytes = chain_bytes = 0;
        dec_has_pred_in = false;
        n_ecb = 0;
    }
};

// Stable grouping of tiles by key index.  A counting sort over the key
// indices in use (one pass to count, one to place; buf is scratch) when they
// are dense enough, else a stable sort.
void group_by_key(std::vector<Unit> &t, std::vector<Unit> &buf) {
    uint32_t max_key = 0;
    for (const Unit &u : t)
        max_key = std::max(max_key, u.meta & META_KEY_MASK);
    const uint64_t n_keys = (uint64_t)max_key + 1;
    if (n_keys > 4 * (uint64_t)t.size() + 64) {
        std::stable_sort(t.begin(), t.end(), [](const Unit &a, const Unit &b) {
            return (a.meta & META_KEY_MASK) < (b.meta & META_KEY_MASK);
        });
        return;
    }
    std::vector<uint64_t> start(n_keys + 1, 0);
    for (const Unit &u : t)
        start[(u.meta & META_KEY_MASK) + 1]++;
    for (uint64_t i = 0; i < n_keys; i++)
        start[i + 1] += start[i];
    buf.resize(t.size());
    for (const Unit &u : t)
        buf[start[u.meta & META_KEY_MASK]++] = u;
    t.swap(buf);
}

// The units of one nonempty request, written from u on; returns the end.
inline Unit *write_request(uint32_t op, uint64_t off, uint64_t len, uint32_t key,
                           const uint8_t *iv, uint32_t tile, Unit *u) {
    const uint32_t meta = key | (op << META_OP_SHIFT);
    if (op == AES_OP_CTR) {
        const uint32_t n0 = le32(iv), n1 = le32(iv + 4);
        uint64_t c = be64(iv + 8);  // mod 2^64, nonce untouched
        for (;; u++) {
            u->off = off;
            u->nbytes = (uint32_t)std::min<uint64_t>(tile, len);
            u->meta = meta;
            u->w[0] = n0;
            u->w[1] = n1;
            u->w[2] = (uint32_t)c;
            u->w[3] = (uint32_t)(c >> 32);
            if (len <= tile)
                return u + 1;
            off += tile;
            len -= tile;
            c += tile / 16;
        }
    }
    u->off = off;
    u->meta = meta;
    if (op == AES_OP_CBC_ENC || op == AES_OP_CBC_DEC)
        memcpy(u->w, iv, 16);
    else
        memset(u->w, 0, 16);  // every block on its own
    if (op == AES_OP_CBC_ENC) {
        u->nbytes = (uint32_t)len;
        return u + 1;
    }
    u->nbytes = (uint32_t)std::min<uint64_t>(tile, len);
    u++;
    const uint32_t next = meta | (op == AES_OP_CBC_DEC ? FLAG_PRED_IN : 0u);
    while (len > tile) {
        off += tile;
        len -= tile;
        u->off = off;
        u->nbytes = (uint32_t)std::min<uint64_t>(tile, len);
        u->meta = next;
        memset(u->w, 0, 16);
        u++;
    }
    return u;
}

// A chain's place in the order "longest first, equal lengths by key index",
// and the request it is.
using ChainKey = std::pair<uint64_t, uint64_t>;

// Sorts a[0, n) by first, requests with the same one in their order (b: room
// for n more); returns where the result is, a or b.  Bytewise, over the bytes
// that differ at all: a batch of equal lengths takes one pass, where a
// comparison sort of 6,542 such chains took 130 us of the host.
ChainKey *sort_chains(ChainKey *a, ChainKey *b, uint64_t n) {
    uint64_t diff = 0;
    bool sorted = true;
    for (uint64_t i = 1; i < n; i++) {
        diff |= a[i].first ^ a[0].first;
        sorted &= a[i - 1].first <= a[i].first;
    }
    for (int shift = 0; shift < 64 && !sorted; shift += 8) {
        if (!((diff >> shift) & 255u))
            continue;
        uint64_t at[256] = {0};
        for (uint64_t i = 0; i < n; i++)
            at[(a[i].first >> shift) & 255u]++;
        uint64_t sum = 0;
        for (uint64_t &v : at) {
            const uint64_t c = v;
            v = sum;
            sum += c;
        }
        for (uint64_t i = 0; i < n; i++)
            b[at[(a[i].first >> shift) & 255u]++] = a[i];
        std::swap(a, b);
    }
    return a;
}

// The unit table of a scanned request list: [CBC- and ECB-decrypt tiles | CTR
// tiles | ECB-encrypt tiles | chains], tiles in request order, chains longest
// first (equal lengths by key index, then in request order): see plan_units.
// keys: room for two entries per chain.
void write_units(const aes_req_t *reqs, uint64_t n, uint32_t tile, const BatchScan &b, Unit *u,
                 ChainKey *keys) {
    Unit *dec = u, *ctr = dec + b.n_dec(), *ecb = ctr + b.units[AES_OP_CTR];
    Unit *chain = dec + b.n_dec() + b.n_enc();
    uint64_t n_chain = 0;
    for (uint64_t i = 0; i < n; i++) {
        const aes_req_t &r = reqs[i];
        if (!r.length)
            continue;
        if (r.op == AES_OP_CBC_ENC) {
            keys[n_chain++] = {(MAX_REQ_BYTES - r.length) / 16 << 32 | r.key_idx, i};
            continue;
        }
        Unit *&w = r.op == AES_OP_CTR ? ctr : r.op == AES_OP_ECB_ENC ? ecb : dec;
        w = write_request(r.op, r.offset, r.length, r.key_idx, r.iv, tile, w);
    }
    const ChainKey *order = sort_chains(keys, keys + n_chain, n_chain);
    for (uint64_t i = 0; i < n_chain; i++) {
        const aes_req_t &r = reqs[order[i].second];
        chain = write_request(r.op, r.offset, r.length, r.key_idx, r.iv, tile, chain);
    }
}

// Cuts every request into units: CTR, ECB and CBC-decrypt into tile_bytes
// tiles (a multiple of 16), CBC-encrypt into one chain each.  p is emptied
// first (its storage kept).  Encryption-side tiles: CTR tiles, then
// ECB-encrypt tiles (the bitsliced kernel takes only the CTR range); with
// group_ctr each of the two groups is ordered by key (request order kept
// within a key), and with group_dec the decryption tiles are, which the
// bitsliced kernels need to share one schedule across a wave's tiles -- the
// table kernels read a schedule per tile.
int plan_units(const aes_req_t *reqs, uint64_t n, uint32_t tile_bytes, bool group_ctr,
               bool group_dec, Planned &p) {
    p.reset();
    try {
        uint64_t n_tiles_ctr = 0, n_tiles_dec = 0, n_chain = 0;
        for (uint64_t i = 0; i < n; i++) {
            const uint64_t t = (reqs[i].length + tile_bytes - 1) / tile_bytes;
            if (is_enc_tile_op(reqs[i].op))
                n_tiles_ctr += t;
            else if (is_dec_tile_op(reqs[i].op))
                n_tiles_dec += t;
            else if (reqs[i].length)
                n_chain++;
        }
        if (n_tiles_ctr >= (1ull << 32) || n_tiles_dec >= (1ull << 32) || n_chain >= (1ull << 32))
            return AES_ERR_RANGE;
        p.ctr.reserve(n_tiles_ctr);
        p.dec.reserve(n_tiles_dec);
        p.chains.reserve(n_chain);
        for (uint64_t i = 0; i < n; i++) {
            const aes_req_t &r = reqs[i];
            if (!r.length)
                continue;
            p.payload += r.length;
            p.extent = std::max(p.extent, r.offset + r.length);
            (r.op == AES_OP_CBC_ENC ? p.chain_bytes
                                    : is_enc_tile_op(r.op) ? p.ctr_bytes : p.dec_bytes) += r.length;
            std::vector<Unit> &v = r.op == AES_OP_CBC_ENC    ? p.chains
                                   : r.op == AES_OP_CTR     ? p.ctr
                                   : r.op == AES_OP_ECB_ENC ? p.ecb
                                                            : p.dec;
            const uint64_t t = r.op == AES_OP_CBC_ENC ? 1 : tile_count(r.length, tile_bytes);
            if (r.op != AES_OP_CBC_ENC)
                p.max_tile = (uint32_t)std::max<uint64_t>(
                    p.max_tile, std::min<uint64_t>(tile_bytes, r.length));
            p.dec_has_pred_in |= r.op == AES_OP_CBC_DEC && t > 1;
            if (r.op != AES_OP_CBC_ENC)
                (is_enc_tile_op(r.op) ? p.enc_work : p.dec_work).sum += TileWork::of(r.length);
            const size_t at = v.size();
            v.resize(at + t);
            write_request(r.op, r.offset, r.length, r.key_idx, r.iv, tile_bytes, v.data() + at);
        }
        if (group_ctr) {
            group_by_key(p.ctr, p.sort_buf);
            group_by_key(p.ecb, p.sort_buf);
        }
        if (group_dec)
            group_by_key(p.dec, p.sort_buf);
        p.n_ecb = p.ecb.size();
        p.ctr.insert(p.ctr.end(), p.ecb.begin(), p.ecb.end());
        // Chains longest first across the batch, so that when there are more
        // chains than chain slots the longest start in the first pass and the
        // batch's makespan is as short as the chains allow; chains of equal
        // length are grouped by key (a wave runs the largest round count
        // among its chains for all of them, so same-key chains share waves).
        std::stable_sort(p.chains.begin(), p.chains.end(), [](const Unit &a, const Unit &b) {
            const uint32_t ka = a.meta & META_KEY_MASK, kb = b.meta & META_KEY_MASK;
            return a.nbytes != b.nbytes ? a.nbytes > b.nbytes : ka < kb;
        });
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    return AES_OK;
}

}  // namespace

// ---------------------------------------------------------------- context

struct Slot {
    void *h_stage = nullptr;  // pinned host staging for the unit table
    void *d_stage = nullptr;  // the device's view of it
    size_t h_cap = 0;
    void *d_units = nullptr;  // device unit table + in-place predecessor snapshots
    size_t d_cap = 0;
    hipEvent_t ev = nullptr;  // recorded after the last launch that used the slot
    bool ev_pending = false;
    hipEvent_t copied = nullptr;  // the unit table's upload on the copy stream
    uint32_t *d_ctrs = nullptr;   // tile-kernel counters: decryption side, then encryption
};

// What a launch reads of its context: the device and the launch configuration.
struct LaunchCtx {
    int device = AES_DEVICE_NONE;
    int n_cu = 0;
    uint32_t *d_timg = nullptr;
    TileLaunch tile_ctr;
    TileLaunch tile_dec;
    ChainLaunch chain{256, 64, true, 0};  // several lanes per chain
    int mixed_nb = 1;        // fused kernel: 1 block per lane (its chain path takes the VGPRs)
    bool fuse = true;        // one launch for batches that mix ops
    int grid = 0;            // tile / fused kernel workgroups, 0 = one per compute unit
    uint32_t ctr_variant = AES_CTR_TABLE;
    uint32_t dec_variant = AES_DEC_TABLE;
};

struct aes_ctx : LaunchCtx {
    char arch[32] = "host";  // device architecture (gcnArchName up to ':'), for the tune cache
    static constexpr int N_SLOTS = 4;
    Slot slots[N_SLOTS];
    int next_slot = 0;
    uint32_t tile_bytes = DEFAULT_TILE;
    hipStream_t capture = nullptr;  // private stream for graph capture and tuning
    // Scratch of the single-call forms, reused from call to call (a context
    // is used by one thread at a time): requests built from the caller's
    // arrays, and the plan of the batch.
    std::vector<aes_req_t> scratch_reqs;
    Planned scratch_plan;
    std::vector<ChainKey> scratch_keys;  // the order of a batch's chains
    std::vector<Unit> scratch_units;     // unit records of a captured call, before their upload
    std::vector<void *> captured;        // tables of captured calls (captured_table)
    size_t captured_bytes = 0;
    std::unique_ptr<HostPool> pool;  // large single-op calls (created on first use)
    hipStream_t copy = nullptr;      // unit-table uploads of the single-call forms
};

struct aes_plan {
    aes_ctx *ctx = nullptr;
    Planned p;
    uint32_t n_scheds = 0;
    uint64_t buf_bytes = 0;
    void *d_units = nullptr;  // [dec | ctr | chains] units, then dec predecessor snapshots
    uint32_t *d_ctrs = nullptr;  // tile-kernel counters: decryption side, then encryption
    size_t n_dec = 0, n_ctr = 0, n_chain = 0;
    uint32_t tile_bytes = DEFAULT_TILE;
};

int aesgpu::ctx_info(const aes_ctx_t *ctx, CtxInfo *out) {
    if (!ctx || !out)
        return AES_ERR_ARG;
    out->device = ctx->device;
    out->n_cu = ctx->n_cu;
    out->d_timg = ctx->d_timg;
    return AES_OK;
}

namespace {

size_t units_bytes(size_t n_dec, size_t n_ctr, size_t n_chain) {
    return (n_dec + n_ctr + n_chain) * sizeof(Unit) + n_dec * 16;
}

struct PlanView {
    const void *d_units;  // unit table, in device memory or in pinned host memory
    void *d_preds;        // in-place predecessor snapshots
    uint32_t *d_ctrs;  // 2 x TILE_CTRS zeroed counters of the tile launches
    size_t n_dec, n_ctr, n_chain;
    bool pred_in;
    uint64_t dec_bytes, ctr_bytes;
    uint64_t chain_bytes;
    uint32_t longest_chain;  // bytes
    uint32_t max_bytes;      // no tile is larger
    TileWork dec_work, enc_work;
    size_t n_ecb;  // ECB-encrypt tiles: the last n_ecb of the n_ctr encryption tiles
    bool zero_ctrs;  // the counters may not be zero: clear what a launch uses first
};

// d_units: the table in device memory, with the snapshots behind it.
PlanView view_of(const Planned &p, void *d_units, uint32_t *d_ctrs) {
    return PlanView{d_units, (Unit *)d_units + (p.dec.size() + p.ctr.size() + p.chains.size()),
                    d_ctrs, p.dec.size(), p.ctr.size(), p.chains.size(), p.dec_has_pred_in,
                    p.dec_bytes, p.ctr_bytes, p.chain_bytes, p.chains.empty() ? 0u : p.chains[0].nbytes,
                    p.max_tile, p.dec_work, p.enc_work, p.n_ecb, false};
}

}  // namespace

// A recorded plan launch, a few recorded request launches, or a HIP graph of
// many.  Few launches are replayed as launches: hipGraphLaunch costs the host
// about 15 us whatever it holds and the device about 6 us around the nodes
// (one request: 15.4 us a replay against 4.0; four: 21.1 against 15.7; a plan
// of two kernels: 38.6 against 31.9), while from eight launches on the graph
// takes less of the host (16.6 us against 25.7) for the same GPU time.
struct aes_graph {
    int device = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    // As captured: the context's configuration, buffers, and either a plan's
    // view or the requests with their tile sizes.
    LaunchCtx cfg;
    const aes_schedule_t *d_scheds = nullptr;
    uint32_t n_scheds = 0;
    const uint8_t *d_in = nullptr;
    uint8_t *d_out = nullptr;
    bool has_plan = false;
    PlanView view{};
    static constexpr uint64_t MAX_DIRECT = 4;
    uint64_t n_reqs = 0;
    aes_req_t reqs[MAX_DIRECT];
    uint32_t tiles[MAX_DIRECT];
};

namespace {

// Zeroed tile-kernel counters for one plan or staging slot (the kernels
// leave them zeroed after every launch).
int alloc_tile_ctrs(uint32_t **out) {
    const size_t bytes = 2 * (size_t)TILE_CTRS * sizeof(uint32_t);
    if (hipMalloc((void **)out, bytes) != hipSuccess) {
        *out = nullptr;
        return AES_ERR_NOMEM;
    }
    const hipError_t e = hipMemset(*out, 0, bytes);
    if (e != hipSuccess) {
        (void)hipFree(*out);
        *out = nullptr;
        return hip_fail(e);
    }
    return AES_OK;
}

// Unit tables of up to this size are read by the kernels straight from the
// pinned staging buffer, larger ones are uploaded.  An upload costs the host a
// copy, an event and a wait (about 15 us a call, 30 us from 256 KiB on);
// reading in place costs the kernel the link's latency and bandwidth (one unit
// 0.5 us, 1,024 units 1.4 us, 4,096 units 4 us, 8,000 to 32,768 units 5 to 7 us
// more than a table in device memory).  At 16,384 tiles of 4 KiB the kernel
// takes 47 us, below what the host spends on such a call with the upload; at
// 32,768 the kernel is the longer part.
constexpr size_t DIRECT_UNITS_BYTES = 16384 * sizeof(Unit);

// Takes the context's next staging slot for a call whose unit table has
// ubytes bytes (need = device bytes with the in-place snapshots): waits for
// the slot's last launch, then grows its pinned and device buffers if needed.
int take_slot(aes_ctx *ctx, size_t ubytes, size_t need, Slot **out) {
    Slot &s = ctx->slots[ctx->next_slot];
    ctx->next_slot = (ctx->next_slot + 1) % aes_ctx::N_SLOTS;
    if (s.ev_pending) {
        HIP_TRY(hipEventSynchronize(s.ev));
        s.ev_pending = false;
    }
    if (s.h_cap < ubytes) {
        if (s.h_stage)
            (void)hipHostFree(s.h_stage);
        s.h_stage = s.d_stage = nullptr;
        s.h_cap = 0;
        if (hipHostMalloc(&s.h_stage, ubytes, hipHostMallocMapped | hipHostMallocCoherent) !=
            hipSuccess)
            return AES_ERR_NOMEM;
        if (hipHostGetDevicePointer(&s.d_stage, s.h_stage, 0) != hipSuccess) {
            (void)hipHostFree(s.h_stage);
            s.h_stage = nullptr;
            return AES_ERR_NOMEM;
        }
        s.h_cap = ubytes;
    }
    if (s.d_cap < need) {
        if (s.d_units)
            (void)hipFree(s.d_units);
        s.d_units = nullptr;
        s.d_cap = 0;
        if (hipMalloc(&s.d_units, need) != hipSuccess)
            return AES_ERR_NOMEM;
        s.d_cap = need;
    }
    if (!s.d_ctrs) {
        const int st = alloc_tile_ctrs(&s.d_ctrs);
        if (st)
            return st;
    }
    *out = &s;
    return AES_OK;
}

// Makes a slot's unit table ready for a launch on `stream` (not being
// captured); *units is where the launch reads it.  A small table is read by the
// kernels from the pinned staging buffer itself.  A larger one is uploaded on
// the context's copy stream and the launch waits for it by event, so the upload
// of one call overlaps the kernels of the call before.  The slot is free of
// earlier uploads and launches (its event was waited for).
int upload_units(aes_ctx *ctx, Slot &s, size_t ubytes, void *stream, const void **units) {
    if (ubytes <= DIRECT_UNITS_BYTES) {
        *units = s.d_stage;
        return AES_OK;
    }
    *units = s.d_units;
    if (!ctx->copy &&
        hipStreamCreateWithFlags(&ctx->copy, hipStreamNonBlocking) != hipSuccess) {
        ctx->copy = nullptr;
        HIP_TRY(hipMemcpyAsync(s.d_units, s.h_stage, ubytes, hipMemcpyHostToDevice,
                               (hipStream_t)stream));
        return AES_OK;
    }
    HIP_TRY(hipMemcpyAsync(s.d_units, s.h_stage, ubytes, hipMemcpyHostToDevice, ctx->copy));
    HIP_TRY(hipEventRecord(s.copied, ctx->copy));
    HIP_TRY(hipStreamWaitEvent((hipStream_t)stream, s.copied, 0));
    return AES_OK;
}

// Whether `stream` is recording into a graph.
int is_capturing(void *stream, bool *out) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing((hipStream_t)stream, &cap));
    *out = cap != hipStreamCaptureStatusNone;
    return AES_OK;
}

// The calling thread may allocate and copy while a stream is being captured
// (on other streams: nothing of it is recorded).
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Device memory that one context holds for the calls it recorded, at most.
constexpr size_t CAPTURED_MAX_BYTES = 4ull << 30;

// The table of a call on a stream that is being captured: device memory of its
// own, filled here once.  A staging slot would not do: replays come after later
// calls have taken the slot again.  The context cannot see how long the graph
// (or an instance of it) lives, so it keeps the table until it is destroyed; a
// graph needs its context anyway, for the cipher tables.
int captured_table(aes_ctx *ctx, const Unit *units, size_t n_units, size_t need, PlanView &v) {
    const size_t ctrs_off = (need + 255) / 256 * 256;
    const size_t bytes = ctrs_off + 2 * (size_t)TILE_CTRS * sizeof(uint32_t);
    if (bytes > CAPTURED_MAX_BYTES - ctx->captured_bytes)
        return AES_ERR_NOMEM;
    try {
        ctx->captured.reserve(ctx->captured.size() + 1);
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    RelaxedCapture relaxed;
    if (!ctx->copy)
        HIP_TRY(hipStreamCreateWithFlags(&ctx->copy, hipStreamNonBlocking));
    uint8_t *d = nullptr;
    if (hipMalloc((void **)&d, bytes) != hipSuccess)
        return AES_ERR_NOMEM;
    ctx->captured.push_back(d);
    ctx->captured_bytes += bytes;
    const int e = launch_zero_words((uint32_t *)(d + ctrs_off), 2 * TILE_CTRS, ctx->copy);
    if (e)
        return hip_fail((hipError_t)e);
    HIP_TRY(hipMemcpyAsync(d, units, n_units * sizeof(Unit), hipMemcpyHostToDevice, ctx->copy));
    HIP_TRY(hipStreamSynchronize(ctx->copy));
    v.d_units = d;
    v.d_preds = (Unit *)d + n_units;
    v.d_ctrs = (uint32_t *)(d + ctrs_off);
    return AES_OK;
}

// Workgroups of the fused kernel that hold the decryption tables: a share of
// the grid proportional to the CBC-decrypt bytes among the parallel bytes.
uint32_t dec_workgroups(const PlanView &v, int grid) {
    if (!v.n_dec)
        return 0;
    if (!v.n_ctr && !v.n_chain)
        return (uint32_t)grid;
    const double share = (double)v.dec_bytes / (double)(v.dec_bytes + v.ctr_bytes + 1);
    long k = std::lround(share * grid);
    if (k < 1)
        k = 1;
    if (k > grid - 1)
        k = grid - 1;
    return (uint32_t)k;
}

// Launches the kernels of one planned batch whose unit table is at v.d_units.
int launch_planned(const LaunchCtx *ctx, const PlanView &v, const aes_schedule_t *d_scheds,
                   uint32_t n_scheds, const uint8_t *d_in, uint8_t *d_out, void *stream) {
    const Unit *u_dec = (const Unit *)v.d_units;
    const Unit *u_ctr = u_dec + v.n_dec;
    const Unit *u_chain = u_ctr + v.n_ctr;
    void *d_preds = nullptr;
    int e;
    if (v.n_dec && v.pred_in && d_in == d_out) {
        d_preds = v.d_preds;
        if ((e = launch_snapshot_preds(u_dec, (uint32_t)v.n_dec, d_in, d_preds, stream)))
            return hip_fail((hipError_t)e);
    }
    // The bitsliced decryption kernel takes every decryption tile in a launch
    // of its own (the predecessor snapshots above included).
    size_t n_dec = v.n_dec;
    if (n_dec && ctx->dec_variant == AES_DEC_BITSLICE) {
        if ((e = launch_dec_bitslice(u_dec, (uint32_t)n_dec, d_scheds, n_scheds, d_preds, d_in,
                                     d_out, stream)))
            return hip_fail((hipError_t)e);
        n_dec = 0;
    }
    // The bitsliced CTR kernel has a launch of its own for the CTR tiles; the
    // table kernels then take only the ECB-encrypt tiles of that range.
    const size_t n_ctr_only = v.n_ctr - v.n_ecb;
    const bool bitslice = ctx->ctr_variant == AES_CTR_BITSLICE && n_ctr_only;
    if (bitslice && (e = launch_ctr_bitslice(u_ctr, (uint32_t)n_ctr_only, d_scheds, n_scheds,
                                             d_in, d_out, ctx->n_cu, stream)))
        return hip_fail((hipError_t)e);
    if (bitslice)
        u_ctr += n_ctr_only;
    const size_t n_ctr_tab = bitslice ? v.n_ecb : v.n_ctr;
    const int kinds = (n_dec > 0) + (n_ctr_tab > 0) + (v.n_chain > 0);
    // One fused launch when CBC-encrypt chains share the batch with tiles: the
    // long chains then run beside the tiles on the workgroups the split gives
    // them.  Without chains, one launch per table set is faster (the tile
    // kernels carry no chain registers).
    if (ctx->fuse && v.n_chain > 0 && kinds > 1) {
        const int grid = ctx->grid > 0 ? ctx->grid : ctx->n_cu;
        MixedArgs a;
        a.dec = u_dec;
        a.ctr = u_ctr;
        a.chains = u_chain;
        a.preds = (const uint32_t *)d_preds;
        a.sched = d_scheds;
        a.timg = ctx->d_timg;
        a.in = d_in;
        a.out = d_out;
        a.n_dec = (uint32_t)n_dec;
        a.n_ctr = (uint32_t)n_ctr_tab;
        a.n_chain = (uint32_t)v.n_chain;
        a.n_sched = n_scheds;
        PlanView fused = v;
        fused.n_dec = n_dec;
        fused.n_ctr = n_ctr_tab;
        fused.ctr_bytes = bitslice ? (v.n_ctr ? v.ctr_bytes * v.n_ecb / v.n_ctr : 0)
                                   : v.ctr_bytes;
        a.n_dec_wg = dec_workgroups(fused, grid);
        a.chain_lanes = (uint32_t)ctx->chain.lanes;
        a.chain_width = (uint32_t)mixed_chain_lanes(
            a.n_chain, v.longest_chain, v.chain_bytes, ctx->chain.quad, (uint32_t)grid - a.n_dec_wg,
            std::max<uint64_t>(fused.ctr_bytes, n_ctr_tab));
        if ((e = launch_mixed(a, ctx->mixed_nb, grid, stream)))
            return hip_fail((hipError_t)e);
        return AES_OK;
    }
    if ((e = launch_cbcdec_tiles(u_dec, (uint32_t)n_dec, v.max_bytes, v.dec_work, d_scheds,
                                 n_scheds, ctx->d_timg, d_preds, d_in, d_out, v.d_ctrs, v.zero_ctrs,
                                 ctx->tile_dec, ctx->n_cu, stream)))
        return hip_fail((hipError_t)e);
    if ((e = launch_ctr_tiles(u_ctr, (uint32_t)n_ctr_tab, v.max_bytes, v.enc_work, d_scheds,
                              n_scheds, ctx->d_timg, d_in, d_out, v.d_ctrs + TILE_CTRS,
                              v.zero_ctrs, ctx->tile_ctr, ctx->n_cu, stream)))
        return hip_fail((hipError_t)e);
    if ((e = launch_cbcenc_chains(u_chain, (uint32_t)v.n_chain, v.longest_chain, v.chain_bytes, d_scheds, n_scheds, ctx->d_timg,
                                  d_in, d_out, ctx->chain, ctx->n_cu, stream)))
        return hip_fail((hipError_t)e);
    return AES_OK;
}

// A few tiles of one side, at `units` in host memory: launched with the unit
// table among the kernel's arguments, so that the call takes no staging buffer,
// copy or event.  False: not such a batch, nothing was launched.
bool launch_few(aes_ctx *ctx, const Unit *units, const PlanView &v, const aes_schedule_t *d_scheds,
                uint32_t n_scheds, const uint8_t *d_in, uint8_t *d_out, void *stream, int *st) {
    const bool dec = v.n_dec > 0;
    if (v.n_chain || (dec && v.n_ctr) || v.n_dec + v.n_ctr > INLINE_UNITS ||
        (v.pred_in && d_in == d_out) || !is_default(dec ? ctx->tile_dec : ctx->tile_ctr) ||
        (dec ? ctx->dec_variant != AES_DEC_TABLE : ctx->ctr_variant != AES_CTR_TABLE))
        return false;
    const hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) {
        *st = hip_fail(e);
        return true;
    }
    int err = hipSuccess;
    if (!launch_tiles_inline(dec, units, (uint32_t)(v.n_dec + v.n_ctr), v.max_bytes, d_scheds,
                             n_scheds, ctx->d_timg, d_in, d_out, ctx->n_cu, stream, &err))
        return false;
    *st = err == hipSuccess ? AES_OK : hip_fail((hipError_t)err);
    return true;
}

void pack_units(const Planned &p, void *dst) {
    Unit *u = (Unit *)dst;
    if (!p.dec.empty())
        memcpy(u, p.dec.data(), p.dec.size() * sizeof(Unit));
    u += p.dec.size();
    if (!p.ctr.empty())
        memcpy(u, p.ctr.data(), p.ctr.size() * sizeof(Unit));
    u += p.ctr.size();
    if (!p.chains.empty())
        memcpy(u, p.chains.data(), p.chains.size() * sizeof(Unit));
}

// Launches a batch of a plan view without its memory: write(u) puts its unit
// records at u.  They go through a staging slot, which is in use until the
// launch is done, or, on a stream that is being captured, into a table of the
// call's own.
template <class Write>
int launch_table(aes_ctx *ctx, PlanView v, const Write &write, const aes_schedule_t *d_scheds,
                 uint32_t n_scheds, const uint8_t *d_in, uint8_t *d_out, void *stream) {
    const size_t n = v.n_dec + v.n_ctr + v.n_chain;
    const size_t need = units_bytes(v.n_dec, v.n_ctr, v.n_chain);
    HIP_TRY(hipSetDevice(ctx->device));
    bool capturing = false;
    int st = is_capturing(stream, &capturing);
    if (st)
        return st;
    if (capturing) {
        try {
            if (ctx->scratch_units.size() < n)
                ctx->scratch_units.resize(n);
        } catch (const std::bad_alloc &) {
            return AES_ERR_NOMEM;
        }
        write(ctx->scratch_units.data());
        if ((st = captured_table(ctx, ctx->scratch_units.data(), n, need, v)))
            return st;
        return launch_planned(ctx, v, d_scheds, n_scheds, d_in, d_out, stream);
    }
    Slot *s = nullptr;
    if ((st = take_slot(ctx, n * sizeof(Unit), need, &s)))
        return st;
    write((Unit *)s->h_stage);
    if ((st = upload_units(ctx, *s, n * sizeof(Unit), stream, &v.d_units)))
        return st;
    v.enc_work.host_table = v.d_units == s->d_stage;
    v.d_preds = (Unit *)s->d_units + n;
    v.d_ctrs = s->d_ctrs;
    st = launch_planned(ctx, v, d_scheds, n_scheds, d_in, d_out, stream);
    // A launch that failed may have started kernels before: the slot is in use
    // until the stream is past them all the same.
    const hipError_t e = hipEventRecord(s->ev, (hipStream_t)stream);
    s->ev_pending = e == hipSuccess;
    if (e != hipSuccess)
        (void)hipStreamSynchronize((hipStream_t)stream);
    return st || e == hipSuccess ? st : hip_fail(e);
}

// A scanned batch as a PlanView without its memory.
PlanView view_of(const BatchScan &b, uint32_t tile) {
    PlanView v{};
    v.n_dec = b.n_dec();
    v.n_ctr = b.n_enc();
    v.n_chain = b.n_chain();
    v.pred_in = b.pred_in;
    v.dec_bytes = b.dec_bytes();
    v.ctr_bytes = b.enc_bytes();
    v.chain_bytes = b.bytes[AES_OP_CBC_ENC];
    v.longest_chain = (uint32_t)b.longest_chain;
    v.max_bytes = (uint32_t)std::min<uint64_t>(tile, b.longest);
    v.dec_work = b.dec_work();
    v.enc_work = b.enc_work();
    v.n_ecb = b.units[AES_OP_ECB_ENC];
    return v;
}

int run_batch(aes_ctx *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
              const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes, const aes_req_t *reqs,
              uint64_t n, void *stream) {
    if (!ctx)
        return AES_ERR_ARG;
    int st = check_buffers(d_in, d_out, buf_bytes, n, d_scheds);
    if (st)
        return st;
    if (n && !reqs)
        return AES_ERR_ARG;
    const uint32_t tile = ctx->tile_bytes;
    BatchScan b;
    if ((st = scan_requests(reqs, n, n_scheds, buf_bytes, tile, b)))
        return st;
    if (!b.ordered) {
        std::vector<std::pair<uint64_t, uint64_t>> ranges;
        try {
            ranges.resize(n);
        } catch (const std::bad_alloc &) {
            return AES_ERR_NOMEM;
        }
        if ((st = check_disjoint(reqs, n, ranges.data())))
            return st;
    }
    PlanView v = view_of(b, tile);
    if (v.n_dec >= (1ull << 32) || v.n_ctr >= (1ull << 32) || v.n_chain >= (1ull << 32))
        return AES_ERR_RANGE;
    const uint64_t n_units = b.n_units();
    if (!n_units)
        return AES_OK;
    // The bitsliced kernels want their tiles grouped by key.
    const bool group_ctr = ctx->ctr_variant == AES_CTR_BITSLICE && v.n_ctr;
    const bool group_dec = ctx->dec_variant == AES_DEC_BITSLICE && v.n_dec;
    Planned &p = ctx->scratch_plan;
    if ((group_ctr || group_dec) &&
        (st = plan_units(reqs, n, tile, group_ctr, group_dec, p)))
        return st;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    if (n_units <= INLINE_UNITS && !v.n_chain) {  // (launch_few takes no chains)
        Unit few[INLINE_UNITS];
        write_units(reqs, n, tile, b, few, nullptr);
        if (launch_few(ctx, few, v, d_scheds, n_scheds, d_in, d_out, stream, &st))
            return st;
    }
    try {
        if (ctx->scratch_keys.size() < 2 * v.n_chain)
            ctx->scratch_keys.resize(2 * v.n_chain);
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    const auto put = [&](Unit *u) {
        if (group_ctr || group_dec)
            pack_units(p, u);
        else
            write_units(reqs, n, tile, b, u, ctx->scratch_keys.data());
    };
    return launch_table(ctx, v, put, d_scheds, n_scheds, d_in, d_out, stream);
}

// ------------------------------------------------- batches without allocation

// aes_batch_noalloc keeps its unit table, in-place predecessor snapshots and
// tile counters in one fixed device array per GPU (`scratch`), and plans on
// the host into fixed static arrays, so that a call allocates nothing.  Its
// device address is taken once per device when a context is created there
// (host code never uses the array's name for device memory).  Every call on a
// device shares that device's array: calls that overlap in time on one device
// (other streams, or other host threads) race on it.
constexpr uint64_t NOALLOC_UNITS_BYTES = (uint64_t)AES_NOALLOC_MAX_UNITS * sizeof(Unit);
constexpr uint64_t NOALLOC_PREDS_BYTES = (uint64_t)AES_NOALLOC_MAX_UNITS * 16;
constexpr uint64_t NOALLOC_CTRS_OFF = NOALLOC_UNITS_BYTES + NOALLOC_PREDS_BYTES;
constexpr uint64_t NOALLOC_SCRATCH_BYTES =
    NOALLOC_CTRS_OFF + 2 * (uint64_t)TILE_CTRS * sizeof(uint32_t);

static __device__ __align__(256) uint8_t scratch[NOALLOC_SCRATCH_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES];  // device address of `scratch`, per device

// Host side of a call: the unit table is built here and copied from here;
// the ranges hold the disjointness check of unsorted requests, then the order
// of the chains (two entries per chain).  Guarded by
// g_noalloc_mu for the whole of a call's host work.
std::mutex g_noalloc_mu;
Unit g_noalloc_units[AES_NOALLOC_MAX_UNITS];
std::pair<uint64_t, uint64_t> g_noalloc_ranges[2 * AES_NOALLOC_MAX_UNITS];

// Takes the device address of `scratch` on the current device (once per
// device).  The caller has made `device` current.
int noalloc_setup(int device) {
    if (device < 0 || device >= NOALLOC_MAX_DEVICES)
        return AES_OK;  // such a device has no scratch; its no-allocation calls fail
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device])
        return AES_OK;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol);
    g_scratch_ptr[device] = p;
    return AES_OK;
}

int run_batch_noalloc(aes_ctx *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                      const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                      const aes_req_t *reqs, uint64_t n, void *stream) {
    if (!ctx)
        return AES_ERR_ARG;
    int st = check_buffers(d_in, d_out, buf_bytes, n, d_scheds);
    if (st)
        return st;
    if (n && !reqs)
        return AES_ERR_ARG;
    // 1. The per-request rules, order, and the unit counts.
    const uint32_t tile = ctx->tile_bytes;
    BatchScan b;
    if ((st = scan_requests(reqs, n, n_scheds, buf_bytes, tile, b)))
        return st;
    const uint64_t n_units = b.n_units();
    if (n_units > AES_NOALLOC_MAX_UNITS)
        return AES_ERR_RANGE;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    // 2. Disjoint output ranges (as many as there are nonempty requests, at
    //    most n_units, where they have to be sorted).
    if (!b.ordered && (st = check_disjoint(reqs, n, g_noalloc_ranges)))
        return st;
    if (!n_units)
        return AES_OK;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    void *d_scratch =
        ctx->device < NOALLOC_MAX_DEVICES ? g_scratch_ptr[ctx->device] : nullptr;
    if (!d_scratch)
        return AES_ERR_DEVICE;
    // 3. Unit records; few of them travel with the launch.
    write_units(reqs, n, tile, b, g_noalloc_units, g_noalloc_ranges);
    PlanView v = view_of(b, tile);
    if (launch_few(ctx, g_noalloc_units, v, d_scheds, n_scheds, d_in, d_out, stream, &st))
        return st;
    // 4. Upload (the static host array is read before the copy call returns,
    //    as for any copy from pageable memory) and launch; a kernel that uses
    //    the tile counters has them cleared first.  A copy that is being
    //    captured would read the array at every replay, after later calls have
    //    written theirs to it: there the records go by value, with kernels.
    HIP_TRY(hipSetDevice(ctx->device));
    bool capturing = false;
    if ((st = is_capturing(stream, &capturing)))
        return st;
    if (capturing) {
        if (const int e = launch_put_units(g_noalloc_units, n_units, d_scratch, stream))
            return hip_fail((hipError_t)e);
    } else {
        HIP_TRY(hipMemcpyAsync(d_scratch, g_noalloc_units, n_units * sizeof(Unit),
                               hipMemcpyHostToDevice, (hipStream_t)stream));
    }
    v.d_units = d_scratch;
    v.d_preds = (Unit *)d_scratch + n_units;
    v.d_ctrs = (uint32_t *)((uint8_t *)d_scratch + NOALLOC_CTRS_OFF);
    v.zero_ctrs = true;
    return launch_planned(ctx, v, d_scheds, n_scheds, d_in, d_out, stream);
}

// ------------------------------------------------- single-op calls over tiles

// Requests per chunk of a single-op call over tiles, and how many threads a
// context has for chunks at most.  (When they are used: launch_rules.h.)
constexpr uint64_t PAR_CHUNK = 4096;
constexpr int PAR_MAX_THREADS = 8;

// Whether the context's threads are there (made on first use).
bool have_pool(aes_ctx *ctx) {
    if (ctx->pool)
        return true;
    const unsigned hw = std::thread::hardware_concurrency();
    const int t = (int)std::min<unsigned>(hw ? hw : 1, PAR_MAX_THREADS);
    try {
        ctx->pool.reset(new HostPool(t - 1));
    } catch (...) {
        return false;
    }
    return true;
}

struct ChunkScan {
    uint64_t err_at = UINT64_MAX;  // first request that breaks a rule
    int err = AES_OK;
    bool ordered = true;  // nonzero requests in offset order and disjoint
    uint64_t first_off = UINT64_MAX, last_end = 0;
    uint64_t tiles = 0, payload = 0, longest = 0, work = 0;
    bool pred_in = false;
};

// The unit records of requests [lo, hi) of a single-op call, from u on.  (Plain
// arguments: in a closure, every store to a record would have them read again.)
void write_single(uint32_t op, const uint64_t *offsets, const uint64_t *lengths,
                  const uint32_t *key_idx, const uint8_t *ivs, uint32_t tile, uint64_t lo,
                  uint64_t hi, Unit *u) {
    for (uint64_t i = lo; i < hi; i++)
        if (lengths[i])
            u = write_request(op, offsets[i], lengths[i], key_idx[i],
                              ivs ? ivs + 16 * i : nullptr, tile, u);
}

// A single-op call over tiles (CBC decryption, CTR, ECB): the requests are
// checked in chunks (on the context's threads if there are many; the rules and
// error precedence of validate), then each chunk writes its unit records
// straight into the pinned staging buffer at offsets from a prefix sum, in
// request order.  Returns 1 when the call is not for this path.
int single_tiles(uint32_t op, aes_ctx *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                 const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                 const uint64_t *offsets, const uint64_t *lengths, const uint32_t *key_idx,
                 const uint8_t *ivs, uint64_t n, void *stream) {
    if (op == AES_OP_CBC_ENC || (op == AES_OP_CTR && ctx->ctr_variant == AES_CTR_BITSLICE) ||
        (is_dec_tile_op(op) && ctx->dec_variant == AES_DEC_BITSLICE) ||
        n / PAR_CHUNK >= (1ull << 30))
        return 1;
    int st = check_buffers(d_in, d_out, buf_bytes, n, d_scheds);
    if (st)
        return st;
    const uint32_t tile = ctx->tile_bytes;
    const bool dec = is_dec_tile_op(op);
    const uint64_t n_chunks = (n + PAR_CHUNK - 1) / PAR_CHUNK;
    const auto run = [&](bool threads, const auto &chunk) {
        if (threads && have_pool(ctx)) {
            ctx->pool->run((int)n_chunks, chunk);
        } else {
            for (uint64_t c = 0; c < n_chunks; c++)
                chunk((int)c);
        }
    };
    std::vector<ChunkScan> sc;
    std::vector<uint64_t> base;
    try {
        sc.resize(n_chunks);
        base.resize(n_chunks + 1);
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    // 1. Rules, order and unit counts per chunk.
    run(scan_in_threads(n), [&](int c) {
        ChunkScan k;
        const uint64_t lo = (uint64_t)c * PAR_CHUNK, hi = std::min(n, lo + PAR_CHUNK);
        for (uint64_t i = lo; i < hi; i++) {
            const uint64_t off = offsets[i], len = lengths[i];
            const int e = check_request(op, off, len, key_idx[i], n_scheds, buf_bytes);
            if (e) {
                k.err_at = i;
                k.err = e;
                break;
            }
            if (!len)
                continue;
            k.ordered &= off >= k.last_end;
            k.first_off = std::min(k.first_off, off);
            k.last_end = std::max(k.last_end, off + len);
            k.tiles += tile_count(len, tile);
            k.payload += len;
            k.work += TileWork::of(len);
            k.longest = std::max(k.longest, len);
        }
        k.pred_in = op == AES_OP_CBC_DEC && k.longest > tile;
        sc[c] = k;
    });
    // 2. The first error in request order, then disjointness.
    uint64_t err_at = UINT64_MAX, payload = 0, longest = 0, work = 0;
    bool ordered = true, pred_in = false;
    uint64_t prev_end = 0;
    base[0] = 0;
    for (uint64_t c = 0; c < n_chunks; c++) {
        if (sc[c].err_at < err_at) {
            err_at = sc[c].err_at;
            st = sc[c].err;
        }
        ordered = ordered && sc[c].ordered &&
                  (sc[c].first_off == UINT64_MAX || sc[c].first_off >= prev_end);
        if (sc[c].first_off != UINT64_MAX)
            prev_end = sc[c].last_end;
        payload += sc[c].payload;
        work += sc[c].work;
        longest = std::max(longest, sc[c].longest);
        pred_in |= sc[c].pred_in;
        base[c + 1] = base[c] + sc[c].tiles;
    }
    if (err_at != UINT64_MAX)
        return st;
    if (!ordered) {  // unsorted (or overlapping): the sort-based check
        std::vector<std::pair<uint64_t, uint64_t>> ranges;
        try {
            ranges.reserve(n);
        } catch (const std::bad_alloc &) {
            return AES_ERR_NOMEM;
        }
        for (uint64_t i = 0; i < n; i++)
            if (lengths[i])
                ranges.emplace_back(offsets[i], offsets[i] + lengths[i]);
        std::sort(ranges.begin(), ranges.end());
        for (size_t i = 1; i < ranges.size(); i++)
            if (ranges[i].first < ranges[i - 1].second)
                return AES_ERR_OVERLAP;
    }
    const uint64_t n_tiles = base[n_chunks];
    if (n_tiles >= (1ull << 32))
        return AES_ERR_RANGE;
    if (!payload)
        return AES_OK;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    PlanView v{};
    v.n_dec = dec ? n_tiles : 0;
    v.n_ctr = dec ? 0 : n_tiles;
    v.pred_in = pred_in;
    v.dec_bytes = dec ? payload : 0;
    v.ctr_bytes = dec ? 0 : payload;
    v.max_bytes = (uint32_t)std::min<uint64_t>(tile, longest);
    (dec ? v.dec_work : v.enc_work).sum = work;
    v.n_ecb = op == AES_OP_ECB_ENC ? n_tiles : 0;
    // 3. Unit records, in request order.
    if (n_tiles <= INLINE_UNITS) {
        Unit few[INLINE_UNITS];
        write_single(op, offsets, lengths, key_idx, ivs, tile, 0, n, few);
        if (launch_few(ctx, few, v, d_scheds, n_scheds, d_in, d_out, stream, &st))
            return st;
    }
    const auto put = [&](Unit *out) {
        run(write_in_threads(n, n_tiles), [&](int c) {
            const uint64_t lo = (uint64_t)c * PAR_CHUNK;
            write_single(op, offsets, lengths, key_idx, ivs, tile, lo, std::min(n, lo + PAR_CHUNK),
                         out + base[c]);
        });
    };
    return launch_table(ctx, v, put, d_scheds, n_scheds, d_in, d_out, stream);
}

int single_mode(uint32_t op, aes_ctx *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes, const uint64_t *offsets,
                const uint64_t *lengths, const uint32_t *key_idx, const uint8_t *ivs, uint64_t n,
                void *stream) {
    if (!ctx)
        return AES_ERR_ARG;
    const bool ecb = op == AES_OP_ECB_ENC || op == AES_OP_ECB_DEC;  // no IVs
    if (n && (!offsets || !lengths || !key_idx || (!ivs && !ecb)))
        return AES_ERR_ARG;
    const int pst = single_tiles(op, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                                 lengths, key_idx, ecb ? nullptr : ivs, n, stream);
    if (pst != 1)
        return pst;
    std::vector<aes_req_t> &reqs = ctx->scratch_reqs;
    try {
        reqs.resize(n);
    } catch (const std::bad_alloc &) {
        return AES_ERR_NOMEM;
    }
    for (uint64_t i = 0; i < n; i++) {
        reqs[i].offset = offsets[i];
        reqs[i].length = lengths[i];
        reqs[i].key_idx = key_idx[i];
        reqs[i].op = op;
        if (ecb)
            memset(reqs[i].iv, 0, 16);
        else
            memcpy(reqs[i].iv, ivs + 16 * i, 16);
    }
    return run_batch(ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, reqs.data(), n, stream);
}

}  // namespace

// ============================================================ exported API

extern "C" {

const char *aes_strerror(int status) {
    switch (status) {
    case AES_OK: return "ok";
    case AES_ERR_ARG: return "invalid argument";
    case AES_ERR_KEYSIZE: return "key size must be 128, 192 or 256 bits";
    case AES_ERR_LENGTH: return "bad length (CBC needs whole 16-byte blocks; requests < 4 GiB)";
    case AES_ERR_RANGE: return "offset, range or key index out of bounds";
    case AES_ERR_OVERLAP: return "requests or buffers overlap";
    case AES_ERR_DEVICE: return "HIP device error or no device";
    case AES_ERR_NOMEM: return "out of memory";
    case AES_ERR_AGAIN: return "resource temporarily unavailable";
    case AES_ERR_TIMEOUT: return "timed out";
    case AES_ERR_STATE: return "invalid state for this call";
    default: return "unknown status";
    }
}

int aes_last_hip_error(void) { return g_last_hip; }

int aes_expand_key(const uint8_t *key, uint32_t key_bits, aes_schedule_t *out) {
    return expand_key(key, key_bits, out);
}

int aes_ctx_create(int hip_device, aes_ctx_t **out) {
    if (!out)
        return AES_ERR_ARG;
    *out = nullptr;
    if (hip_device < AES_DEVICE_NONE)
        return AES_ERR_ARG;
    aes_ctx *ctx = new (std::nothrow) aes_ctx();
    if (!ctx)
        return AES_ERR_NOMEM;
    ctx->device = hip_device;
    if (hip_device != AES_DEVICE_NONE) {
        int ndev = 0;
        hipError_t e = hipGetDeviceCount(&ndev);
        if (e != hipSuccess || hip_device >= ndev) {
            delete ctx;
            return hip_fail(e != hipSuccess ? e : hipErrorInvalidDevice);
        }
        hipDeviceProp_t prop;
        if ((e = hipSetDevice(hip_device)) != hipSuccess ||
            (e = hipGetDeviceProperties(&prop, hip_device)) != hipSuccess) {
            delete ctx;
            return hip_fail(e);
        }
        ctx->n_cu = prop.multiProcessorCount;
        size_t an = strcspn(prop.gcnArchName, ":");
        an = an < sizeof(ctx->arch) - 1 ? an : sizeof(ctx->arch) - 1;
        memcpy(ctx->arch, prop.gcnArchName, an);
        ctx->arch[an] = '\0';
        uint32_t img[TIMG_WORDS];
        make_table_image(img);
        if (hipMalloc((void **)&ctx->d_timg, sizeof(img)) != hipSuccess) {
            delete ctx;
            return AES_ERR_NOMEM;
        }
        if ((e = hipMemcpy(ctx->d_timg, img, sizeof(img), hipMemcpyHostToDevice)) != hipSuccess) {
            (void)hipFree(ctx->d_timg);
            delete ctx;
            return hip_fail(e);
        }
        if (int st = noalloc_setup(hip_device)) {
            (void)hipFree(ctx->d_timg);
            delete ctx;
            return st;
        }
        for (Slot &s : ctx->slots) {
            if ((e = hipEventCreateWithFlags(&s.ev, hipEventDisableTiming)) != hipSuccess ||
                (e = hipEventCreateWithFlags(&s.copied, hipEventDisableTiming)) != hipSuccess) {
                aes_ctx_destroy(ctx);
                return hip_fail(e);
            }
        }
    }
    *out = ctx;
    return AES_OK;
}

void aes_ctx_destroy(aes_ctx_t *ctx) {
    if (!ctx)
        return;
    if (ctx->device != AES_DEVICE_NONE) {
        (void)hipSetDevice(ctx->device);
        for (Slot &s : ctx->slots) {
            if (s.ev) {
                if (s.ev_pending)
                    (void)hipEventSynchronize(s.ev);
                (void)hipEventDestroy(s.ev);
            }
            if (s.copied)
                (void)hipEventDestroy(s.copied);
            if (s.h_stage)
                (void)hipHostFree(s.h_stage);
            if (s.d_units)
                (void)hipFree(s.d_units);
            if (s.d_ctrs)
                (void)hipFree(s.d_ctrs);
        }
        for (void *d : ctx->captured)
            (void)hipFree(d);
        if (ctx->d_timg)
            (void)hipFree(ctx->d_timg);
        if (ctx->capture)
            (void)hipStreamDestroy(ctx->capture);
        if (ctx->copy) {
            (void)hipStreamSynchronize(ctx->copy);
            (void)hipStreamDestroy(ctx->copy);
        }
    }
    delete ctx;
}

int aes_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
              const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes, const aes_req_t *reqs,
              uint64_t n_reqs, void *stream) {
    return run_batch(ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, reqs, n_reqs, stream);
}

int aes_batch_noalloc(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                      const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                      const aes_req_t *reqs, uint64_t n_reqs, void *stream) {
    return run_batch_noalloc(ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, reqs, n_reqs,
                             stream);
}

int aes_cbc_encrypt_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                          const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                          const uint64_t *offsets, const uint64_t *lengths,
                          const uint32_t *key_idx, const uint8_t *ivs, uint64_t n, void *stream) {
    return single_mode(AES_OP_CBC_ENC, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                       lengths, key_idx, ivs, n, stream);
}

int aes_cbc_decrypt_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                          const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                          const uint64_t *offsets, const uint64_t *lengths,
                          const uint32_t *key_idx, const uint8_t *ivs, uint64_t n, void *stream) {
    return single_mode(AES_OP_CBC_DEC, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                       lengths, key_idx, ivs, n, stream);
}

int aes_ctr_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                  const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                  const uint64_t *offsets, const uint64_t *lengths, const uint32_t *key_idx,
                  const uint8_t *ivs, uint64_t n, void *stream) {
    return single_mode(AES_OP_CTR, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                       lengths, key_idx, ivs, n, stream);
}

int aes_ecb_encrypt_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                          const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                          const uint64_t *offsets, const uint64_t *lengths,
                          const uint32_t *key_idx, const uint8_t *ivs, uint64_t n,
                          void *stream) {
    return single_mode(AES_OP_ECB_ENC, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                       lengths, key_idx, ivs, n, stream);
}

int aes_ecb_decrypt_batch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                          const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                          const uint64_t *offsets, const uint64_t *lengths,
                          const uint32_t *key_idx, const uint8_t *ivs, uint64_t n,
                          void *stream) {
    return single_mode(AES_OP_ECB_DEC, ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, offsets,
                       lengths, key_idx, ivs, n, stream);
}

// ------------------------------------------------------------------ plans

int aes_plan_create(aes_ctx_t *ctx, const aes_req_t *reqs, uint64_t n, uint32_t n_scheds,
                    uint64_t buf_bytes, aes_plan_t **out) {
    if (!ctx || !out)
        return AES_ERR_ARG;
    *out = nullptr;
    int st = validate(reqs, n, n_scheds, buf_bytes);
    if (st)
        return st;
    aes_plan *pl = new (std::nothrow) aes_plan();
    if (!pl)
        return AES_ERR_NOMEM;
    pl->ctx = ctx;
    pl->tile_bytes = ctx->tile_bytes;
    pl->n_scheds = n_scheds;
    pl->buf_bytes = buf_bytes;
    if ((st = plan_units(reqs, n, ctx->tile_bytes, ctx->ctr_variant == AES_CTR_BITSLICE,
                         ctx->dec_variant == AES_DEC_BITSLICE, pl->p))) {
        delete pl;
        return st;
    }
    pl->n_dec = pl->p.dec.size();
    pl->n_ctr = pl->p.ctr.size();
    pl->n_chain = pl->p.chains.size();
    if (ctx->device != AES_DEVICE_NONE && pl->p.payload) {
        hipError_t e;
        const size_t need = units_bytes(pl->n_dec, pl->n_ctr, pl->n_chain);
        const size_t ubytes = (pl->n_dec + pl->n_ctr + pl->n_chain) * sizeof(Unit);
        std::vector<Unit> host;
        try {
            host.resize(pl->n_dec + pl->n_ctr + pl->n_chain);
        } catch (const std::bad_alloc &) {
            delete pl;
            return AES_ERR_NOMEM;
        }
        pack_units(pl->p, host.data());
        if ((e = hipSetDevice(ctx->device)) != hipSuccess) {
            delete pl;
            return hip_fail(e);
        }
        if (hipMalloc(&pl->d_units, need) != hipSuccess) {
            delete pl;
            return AES_ERR_NOMEM;
        }
        if ((e = hipMemcpy(pl->d_units, host.data(), ubytes, hipMemcpyHostToDevice)) !=
            hipSuccess) {
            (void)hipFree(pl->d_units);
            delete pl;
            return hip_fail(e);
        }
        if ((st = alloc_tile_ctrs(&pl->d_ctrs))) {
            (void)hipFree(pl->d_units);
            delete pl;
            return st;
        }
    }
    *out = pl;
    return AES_OK;
}

int aes_plan_launch(aes_plan_t *plan, const aes_schedule_t *d_scheds, const uint8_t *d_in,
                    uint8_t *d_out, void *stream) {
    if (!plan)
        return AES_ERR_ARG;
    const uint64_t n = plan->n_dec + plan->n_ctr + plan->n_chain;
    int st = check_buffers(d_in, d_out, plan->buf_bytes, n, d_scheds);
    if (st)
        return st;
    if (!plan->p.payload)
        return AES_OK;
    aes_ctx *ctx = plan->ctx;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    HIP_TRY(hipSetDevice(ctx->device));
    return launch_planned(ctx, view_of(plan->p, plan->d_units, plan->d_ctrs),
                          d_scheds, plan->n_scheds, d_in, d_out, stream);
}

int aes_plan_info(const aes_plan_t *plan, aes_plan_info_t *info) {
    if (!plan || !info)
        return AES_ERR_ARG;
    memset(info, 0, sizeof(*info));
    info->n_units_cbc_dec = plan->n_dec;
    info->n_units_ctr = plan->n_ctr;
    info->n_chains_cbc_enc = plan->n_chain;
    info->payload_bytes = plan->p.payload;
    info->extent_bytes = plan->p.extent;
    info->tile_bytes = plan->tile_bytes;
    return AES_OK;
}

int aes_plan_units(const aes_plan_t *plan, aes_unit_t *out, uint64_t max, uint64_t *n_out) {
    if (!plan || !n_out || (max && !out))
        return AES_ERR_ARG;
    static_assert(sizeof(aes_unit_t) == sizeof(Unit), "unit record layout");
    const uint64_t total = plan->n_dec + plan->n_ctr + plan->n_chain;
    *n_out = total;
    uint64_t k = 0;
    for (const auto *v : {&plan->p.dec, &plan->p.ctr, &plan->p.chains})
        for (const Unit &u : *v) {
            if (k >= max)
                return AES_OK;
            memcpy(&out[k++], &u, sizeof(Unit));
        }
    return AES_OK;
}

void aes_plan_destroy(aes_plan_t *plan) {
    if (!plan)
        return;
    if (plan->d_units || plan->d_ctrs) {
        (void)hipSetDevice(plan->ctx->device);
        (void)hipDeviceSynchronize();
        if (plan->d_units)
            (void)hipFree(plan->d_units);
        if (plan->d_ctrs)
            (void)hipFree(plan->d_ctrs);
    }
    delete plan;
}

// ----------------------------------------------------------- launch config

int aes_ctx_get_config(const aes_ctx_t *ctx, aes_launch_config_t *cfg) {
    if (!ctx || !cfg)
        return AES_ERR_ARG;
    memset(cfg, 0, sizeof(*cfg));
    cfg->tile_bytes = ctx->tile_bytes;
    cfg->ctr_nb = (uint32_t)ctx->tile_ctr.nb;
    cfg->ctr_wg = (uint32_t)ctx->tile_ctr.wg_threads;
    cfg->dec_nb = (uint32_t)ctx->tile_dec.nb;
    cfg->dec_wg = (uint32_t)ctx->tile_dec.wg_threads;
    cfg->chain_lanes = (uint32_t)ctx->chain.lanes;
    cfg->chain_wg = (uint32_t)ctx->chain.wg_threads;
    cfg->chain_quad = ctx->chain.quad ? 1u : 0u;
    cfg->mixed_nb = (uint32_t)ctx->mixed_nb;
    cfg->fuse = ctx->fuse ? 1u : 0u;
    cfg->grid = (uint32_t)ctx->grid;
    cfg->ctr_variant = ctx->ctr_variant;
    cfg->dec_variant = ctx->dec_variant;
    return AES_OK;
}

int aes_ctx_set_config(aes_ctx_t *ctx, const aes_launch_config_t *cfg) {
    if (!ctx || !cfg)
        return AES_ERR_ARG;
    if (cfg->tile_bytes < 1024 || cfg->tile_bytes > (1u << 24) || (cfg->tile_bytes & 1023))
        return AES_ERR_ARG;
    if (!tile_shape_supported((int)cfg->ctr_nb, (int)cfg->ctr_wg) ||
        !tile_shape_supported((int)cfg->dec_nb, (int)cfg->dec_wg))
        return AES_ERR_ARG;
    if (cfg->chain_lanes < 1 || cfg->chain_lanes > 64 || cfg->chain_wg < 64 ||
        cfg->chain_wg > 1024 || (cfg->chain_wg & 63))
        return AES_ERR_ARG;
    if (cfg->mixed_nb != 1 && cfg->mixed_nb != 2)
        return AES_ERR_ARG;
    if (cfg->fuse > 1 || cfg->grid > 65535)
        return AES_ERR_ARG;
    if (cfg->ctr_variant != AES_CTR_TABLE && cfg->ctr_variant != AES_CTR_BITSLICE)
        return AES_ERR_ARG;
    if (cfg->dec_variant != AES_DEC_TABLE && cfg->dec_variant != AES_DEC_BITSLICE)
        return AES_ERR_ARG;
    if (cfg->chain_quad > 1)
        return AES_ERR_ARG;
    ctx->tile_bytes = cfg->tile_bytes;
    ctx->tile_ctr.nb = (int)cfg->ctr_nb;
    ctx->tile_ctr.wg_threads = (int)cfg->ctr_wg;
    ctx->tile_ctr.grid = (int)cfg->grid;
    ctx->tile_dec.nb = (int)cfg->dec_nb;
    ctx->tile_dec.wg_threads = (int)cfg->dec_wg;
    ctx->tile_dec.grid = (int)cfg->grid;
    ctx->chain.lanes = (int)cfg->chain_lanes;
    ctx->chain.wg_threads = (int)cfg->chain_wg;
    ctx->chain.quad = cfg->chain_quad != 0;
    ctx->mixed_nb = (int)cfg->mixed_nb;
    ctx->fuse = cfg->fuse != 0;
    ctx->grid = (int)cfg->grid;
    ctx->ctr_variant = cfg->ctr_variant;
    ctx->dec_variant = cfg->dec_variant;
    return AES_OK;
}

// ---------------------------------------------------- one request, one launch

namespace {

// Bytes per unit of a request's own launch, where the kernel for short ones does
// not take it.  In place, a multi-tile CBC decryption then stays in one wave,
// which carries each predecessor block in registers before overwriting it.
uint32_t request_tile(const aes_ctx *ctx, const aes_req_t &r, bool in_place) {
    return r.op == AES_OP_CBC_DEC && in_place && r.length > ctx->tile_bytes ? (uint32_t)r.length
                                                                            : ctx->tile_bytes;
}

}  // namespace

int aes_request_launch(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                       const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                       const aes_req_t *req, void *stream) {
    if (!ctx || !req)
        return AES_ERR_ARG;
    int st = check_buffers(d_in, d_out, buf_bytes, 1, d_scheds);
    if (st)
        return st;
    if ((st = validate(req, 1, n_scheds, buf_bytes)))
        return st;
    if (!req->length)
        return AES_OK;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    HIP_TRY(hipSetDevice(ctx->device));
    const int e = launch_request(*req, request_tile(ctx, *req, d_in == d_out), d_scheds, n_scheds,
                                 ctx->d_timg, d_in, d_out,
                                 ctx->n_cu, stream);
    if (e)
        return hip_fail((hipError_t)e);
    return AES_OK;
}

int aes_request_launches(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                         const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                         const aes_req_t *reqs, uint64_t n_reqs, void *stream) {
    if (!ctx)
        return AES_ERR_ARG;
    int st = check_buffers(d_in, d_out, buf_bytes, n_reqs, d_scheds);
    if (st)
        return st;
    if ((st = validate(reqs, n_reqs, n_scheds, buf_bytes)))
        return st;
    for (uint64_t i = 0; i < n_reqs && !st; i++)
        st = aes_request_launch(ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, &reqs[i],
                                stream);
    return st;
}

// -------------------------------------------------------------- HIP graphs

namespace {

int capture_stream(aes_ctx *ctx) {
    if (!ctx->capture)
        HIP_TRY(hipStreamCreateWithFlags(&ctx->capture, hipStreamNonBlocking));
    return AES_OK;
}

// A graph record of launches on the context's device over these buffers.
aes_graph *new_graph(const aes_ctx *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                     const uint8_t *d_in, uint8_t *d_out) {
    aes_graph *g = new (std::nothrow) aes_graph();
    if (!g)
        return nullptr;
    g->device = ctx->device;
    g->cfg = *ctx;
    g->d_scheds = d_scheds;
    g->n_scheds = n_scheds;
    g->d_in = d_in;
    g->d_out = d_out;
    return g;
}

}  // namespace

int aes_plan_graph(aes_plan_t *plan, const aes_schedule_t *d_scheds, const uint8_t *d_in,
                   uint8_t *d_out, aes_graph_t **out) {
    if (!plan || !out)
        return AES_ERR_ARG;
    *out = nullptr;
    aes_ctx *ctx = plan->ctx;
    const uint64_t n = plan->n_dec + plan->n_ctr + plan->n_chain;
    int st = check_buffers(d_in, d_out, plan->buf_bytes, n, d_scheds);
    if (st)
        return st;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    aes_graph *g = new_graph(ctx, d_scheds, plan->n_scheds, d_in, d_out);
    if (!g)
        return AES_ERR_NOMEM;
    g->has_plan = plan->p.payload != 0;
    g->view = view_of(plan->p, plan->d_units, plan->d_ctrs);
    *out = g;
    return AES_OK;
}

int aes_requests_graph(aes_ctx_t *ctx, const aes_schedule_t *d_scheds, uint32_t n_scheds,
                       const uint8_t *d_in, uint8_t *d_out, uint64_t buf_bytes,
                       const aes_req_t *reqs, uint64_t n_reqs, aes_graph_t **out) {
    if (!ctx || !out)
        return AES_ERR_ARG;
    *out = nullptr;
    int st = check_buffers(d_in, d_out, buf_bytes, n_reqs, d_scheds);
    if (st)
        return st;
    if ((st = validate(reqs, n_reqs, n_scheds, buf_bytes)))
        return st;
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    HIP_TRY(hipSetDevice(ctx->device));
    aes_graph *g = new_graph(ctx, d_scheds, n_scheds, d_in, d_out);
    if (!g)
        return AES_ERR_NOMEM;
    uint64_t live = 0;
    for (uint64_t i = 0; i < n_reqs; i++)
        live += reqs[i].length != 0;
    if (live <= aes_graph::MAX_DIRECT) {
        for (uint64_t i = 0; i < n_reqs; i++) {
            if (!reqs[i].length)
                continue;
            g->reqs[g->n_reqs] = reqs[i];
            g->tiles[g->n_reqs++] = request_tile(ctx, reqs[i], d_in == d_out);
        }
        *out = g;
        return AES_OK;
    }
    if ((st = capture_stream(ctx))) {
        aes_graph_destroy(g);
        return st;
    }
    hipError_t e = hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        for (uint64_t i = 0; i < n_reqs && !st; i++) {
            if (reqs[i].length)
                st = aes_request_launch(ctx, d_scheds, n_scheds, d_in, d_out, buf_bytes, &reqs[i],
                                        ctx->capture);
        }
        e = hipStreamEndCapture(ctx->capture, &g->graph);
        if (!st && e == hipSuccess)
            e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    }
    if (!st && e != hipSuccess)
        st = hip_fail(e);
    if (st) {
        aes_graph_destroy(g);
        return st;
    }
    *out = g;
    return AES_OK;
}

int aes_graph_launch(aes_graph_t *g, void *stream) {
    if (!g)
        return AES_ERR_ARG;
    HIP_TRY(hipSetDevice(g->device));
    if (g->exec) {
        HIP_TRY(hipGraphLaunch(g->exec, (hipStream_t)stream));
        return AES_OK;
    }
    if (g->has_plan)
        return launch_planned(&g->cfg, g->view, g->d_scheds, g->n_scheds, g->d_in, g->d_out,
                              stream);
    for (uint64_t i = 0; i < g->n_reqs; i++) {
        const int e = launch_request(g->reqs[i], g->tiles[i], g->d_scheds, g->n_scheds,
                                     g->cfg.d_timg, g->d_in, g->d_out, g->cfg.n_cu, stream);
        if (e)
            return hip_fail((hipError_t)e);
    }
    return AES_OK;
}

void aes_graph_destroy(aes_graph_t *g) {
    if (!g)
        return;
    (void)hipSetDevice(g->device);
    if (g->exec)
        (void)hipGraphExecDestroy(g->exec);
    if (g->graph)
        (void)hipGraphDestroy(g->graph);
    delete g;
}

// ----------------------------------------------------------------- tuning

namespace {

// Median time in ms of `iters` launches of plan (after one warm-up).
int time_plan(aes_plan *plan, const aes_schedule_t *d_scheds, const uint8_t *d_in,
              uint8_t *d_out, int iters, double *ms_out) {
    aes_ctx *ctx = plan->ctx;
    hipEvent_t a, b;
    HIP_TRY(hipEventCreate(&a));
    HIP_TRY(hipEventCreate(&b));
    std::vector<double> ms;
    int st = AES_OK;
    for (int i = 0; i <= iters && !st; i++) {
        hipError_t e = hipEventRecord(a, ctx->capture);
        if (e == hipSuccess) {
            st = launch_planned(ctx,
                                view_of(plan->p, plan->d_units, plan->d_ctrs),
                                d_scheds, plan->n_scheds, d_in, d_out, ctx->capture);
            if (!st)
                e = hipEventRecord(b, ctx->capture);
        }
        if (!st && e == hipSuccess)
            e = hipEventSynchronize(b);
        if (!st && e != hipSuccess)
            st = hip_fail(e);
        float t = 0.f;
        if (!st && (e = hipEventElapsedTime(&t, a, b)) != hipSuccess)
            st = hip_fail(e);
        if (!st && i > 0)
            ms.push_back(t);
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (st)
        return st;
    std::sort(ms.begin(), ms.end());
    *ms_out = ms[ms.size() / 2];
    return AES_OK;
}

}  // namespace

// Relative gain a tuning candidate needs to replace the best so far.
constexpr double TUNE_MARGIN = 0.02;

int aes_tune(aes_ctx_t *ctx, const aes_req_t *reqs, uint64_t n_reqs, uint32_t n_scheds,
             uint64_t buf_bytes, const aes_schedule_t *d_scheds, const uint8_t *d_in,
             uint8_t *d_out, uint32_t iters, aes_launch_config_t *best_out) {
    if (!ctx || (n_reqs && !reqs) || iters < 1 || iters > 1000)
        return AES_ERR_ARG;
    int st = check_buffers(d_in, d_out, buf_bytes, n_reqs, d_scheds);
    if (st)
        return st;
    if (n_reqs && d_in == d_out)
        return AES_ERR_OVERLAP;  // repeated runs must not feed on their own output
    if ((st = validate(reqs, n_reqs, n_scheds, buf_bytes)))
        return st;
    // The tune cache: a stored configuration for a batch of this shape is
    // applied without timing (if the library still supports it).
    const char *cache = getenv("AESGPU_TUNE_CACHE");
    std::string sig;
    if (cache && *cache) {
        sig = tune_signature(ctx->arch, ctx->n_cu, reqs, n_reqs, n_scheds);
        aes_launch_config_t c;
        // The cache holds the tuned knobs; the decryption variant is the
        // caller's and stays as set.
        if (tune_cache_lookup(cache, sig, &c) && ((c.dec_variant = ctx->dec_variant), true) &&
            aes_ctx_set_config(ctx, &c) == AES_OK) {
            if (best_out)
                aes_ctx_get_config(ctx, best_out);
            return AES_OK;
        }
    }
    if (ctx->device == AES_DEVICE_NONE)
        return AES_ERR_DEVICE;
    HIP_TRY(hipSetDevice(ctx->device));
    if ((st = capture_stream(ctx)))
        return st;
    aes_launch_config_t best;
    aes_ctx_get_config(ctx, &best);
    double best_ms = 1e30;
    // One candidate: set it, (re)plan when the tile size or the CTR variant
    // (which decides the key grouping of CTR tiles) changed, time it.
    aes_plan *plan = nullptr;
    uint32_t plan_tile = 0, plan_variant = 0;
    auto trial = [&](const aes_launch_config_t &c) -> int {
        int s2 = aes_ctx_set_config(ctx, &c);
        if (s2)
            return AES_OK;  // shape not available: skip
        if (!plan || plan_tile != c.tile_bytes || plan_variant != c.ctr_variant) {
            aes_plan_destroy(plan);
            plan = nullptr;
            if ((s2 = aes_plan_create(ctx, reqs, n_reqs, n_scheds, buf_bytes, &plan)))
                return s2;
            plan_tile = c.tile_bytes;
            plan_variant = c.ctr_variant;
        }
        double ms = 0;
        if ((s2 = time_plan(plan, d_scheds, d_in, d_out, (int)iters, &ms)))
            return s2;
        // A candidate must beat the best by more than run-to-run noise: where
        // a knob does not matter (a batch bound by one long CBC-enc chain
        // times the same under every tile shape) the starting value stays,
        // instead of whichever shape a timing fluctuation favoured.
        if (ms < best_ms * (1.0 - TUNE_MARGIN)) {
            best_ms = ms;
            best = c;
        }
        return AES_OK;
    };
    // Coordinate descent from the starting configuration, one knob at a time
    // from the best point so far, and only over knobs the batch's launch uses
    // (a knob the launch ignores would be set by timing noise alone): tile
    // size; the fusion switch (batches mixing CBC-encrypt chains with tiles);
    // tile-kernel shapes (unfused launches with tiles); the fused kernel's
    // blocks per lane (fused launches); chain mode (batches with chains); the
    // CTR variant (batches with CTR requests).
    aes_launch_config_t c = best;
    st = trial(c);
    if (!st && !plan)
        st = AES_ERR_ARG;  // the context's own configuration did not apply
    if (st) {
        aes_plan_destroy(plan);
        (void)aes_ctx_set_config(ctx, &best);
        return st;
    }
    // Which unit kinds the batch has (the plan is rebuilt by later trials;
    // only whether each kind is present is kept, which no knob changes).
    const bool has_dec = !plan->p.dec.empty();
    const bool has_ctr = plan->p.ctr.size() > plan->p.n_ecb;
    const bool has_ecb_enc = plan->p.n_ecb > 0;
    const bool has_chains = !plan->p.chains.empty();
    const bool has_tiles = has_dec || has_ctr || has_ecb_enc;
    // Whether the table tile kernels run, and whether one fused launch takes
    // the batch, under k (as launch_planned decides: the bitsliced variant
    // launches the CTR tiles on their own).
    auto table_tiles = [&](const aes_launch_config_t &k) {
        return (has_dec && k.dec_variant != AES_DEC_BITSLICE) || has_ecb_enc ||
               (has_ctr && k.ctr_variant != AES_CTR_BITSLICE);
    };
    auto fused = [&](const aes_launch_config_t &k) {
        const bool ctr_tab = has_ecb_enc || (has_ctr && k.ctr_variant != AES_CTR_BITSLICE);
        const bool dec_tab = has_dec && k.dec_variant != AES_DEC_BITSLICE;
        const int kinds = (int)dec_tab + (int)ctr_tab + (int)has_chains;
        return k.fuse && has_chains && kinds > 1;
    };
    const uint32_t tiles[] = {4096, 8192, 16384};
    for (uint32_t t : tiles) {
        if (st || !has_tiles)
            break;
        c = best;
        c.tile_bytes = t;
        st = trial(c);
    }
    for (uint32_t f = 0; f <= 1 && !st && has_chains && has_tiles; f++) {
        c = best;
        c.fuse = f;
        st = trial(c);
    }
    const uint32_t shapes[][2] = {{1, 1024}, {2, 1024}, {2, 512}, {4, 512}, {4, 256}, {1, 512}};
    for (auto &sh : shapes) {
        if (st || fused(best) || !table_tiles(best))
            break;
        c = best;
        c.ctr_nb = c.dec_nb = sh[0];
        c.ctr_wg = c.dec_wg = sh[1];
        st = trial(c);
    }
    for (uint32_t mnb = 1; mnb <= 2 && !st && fused(best); mnb++) {
        c = best;
        c.mixed_nb = mnb;
        st = trial(c);
    }
    const uint32_t lanes[] = {16, 32, 64};
    for (uint32_t l : lanes) {
        if (st || !has_chains)
            break;
        c = best;
        c.chain_lanes = l;
        c.chain_quad = 0;
        st = trial(c);
    }
    if (!st && has_chains) {  // several lanes per chain
        c = best;
        c.chain_quad = 1;
        st = trial(c);
    }
    for (uint32_t v = AES_CTR_TABLE; v <= AES_CTR_BITSLICE && has_ctr && !st; v++) {
        c = best;
        c.ctr_variant = v;
        st = trial(c);
    }
    aes_plan_destroy(plan);
    (void)aes_ctx_set_config(ctx, &best);
    if (st)
        return st;
    if (cache && *cache)
        (void)tune_cache_store(cache, sig, best);  // a cache that cannot be written is skipped
    if (best_out)
        *best_out = best;
    return AES_OK;
}

int aes_host_batch(const aes_schedule_t *scheds, uint32_t n_scheds, const uint8_t *in,
                   uint8_t *out, uint64_t buf_bytes, const aes_req_t *reqs, uint64_t n_reqs,
                   uint32_t n_threads) {
    if (n_threads > 1024)
        return AES_ERR_ARG;
    int st = check_buffers(in, out, buf_bytes, n_reqs, scheds);
    if (st)
        return st;
    if ((st = validate(reqs, n_reqs, n_scheds, buf_bytes)))
        return st;
    if (!n_reqs)
        return AES_OK;
    uint64_t nt = n_threads;
    if (!nt) {  // the CPUs this process may run on (a machine may have more)
        cpu_set_t set;
        nt = sched_getaffinity(0, sizeof(set), &set) == 0 ? (uint64_t)CPU_COUNT(&set)
                                                          : std::thread::hardware_concurrency();
    }
    nt = std::max<uint64_t>(1, std::min<uint64_t>(nt, n_reqs));
    // Requests are claimed one at a time (their sizes differ; k at a time
    // only past 2^31 requests).  The error reported is the one of the
    // lowest-numbered request that failed; the others still run.
    const uint64_t k = (n_reqs + INT32_MAX - 1) / INT32_MAX;
    std::mutex m;
    uint64_t bad_i = UINT64_MAX;
    int bad_code = AES_OK;
    HostPool pool((int)nt - 1);
    pool.run((int)((n_reqs + k - 1) / k), [&](int c) {
        const uint64_t end = std::min<uint64_t>(n_reqs, ((uint64_t)c + 1) * k);
        for (uint64_t i = (uint64_t)c * k; i < end; i++) {
            const aes_req_t &r = reqs[i];
            const int e = aes_host_route_crypt(&scheds[r.key_idx], r.op, r.iv, in + r.offset,
                                               out + r.offset, r.length);
            if (e) {
                std::lock_guard<std::mutex> lk(m);
                if (i < bad_i) {
                    bad_i = i;
                    bad_code = e;
                }
            }
        }
    });
    return bad_code;
}

int aes_tune_key(const aes_ctx_t *ctx, const aes_req_t *reqs, uint64_t n_reqs, uint32_t n_scheds,
                 char *buf, size_t cap, size_t *len_out) {
    if (!ctx || (n_reqs && !reqs) || (cap && !buf))
        return AES_ERR_ARG;
    const std::string sig = tune_signature(ctx->arch, ctx->n_cu, reqs, n_reqs, n_scheds);
    if (len_out)
        *len_out = sig.size();
    if (cap < sig.size() + 1)
        return AES_ERR_ARG;
    memcpy(buf, sig.c_str(), sig.size() + 1);
    return AES_OK;
}

}  // extern "C"
