// Host side of libpbkv: argument validation, work-list construction and launches behind
// the C boundary declared in include/pbkv.h.  No attention, append or swap-in arithmetic
// happens on the host: the host only cuts the batch into tiles / page runs and enqueues
// the kernels.
#include "../../include/pbkv.h"
#include "pbkv_internal.h"

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

}  // namespace

// error text for the translation units that hold no HIP code (the policy core)
int pbkv::set_error(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}
void pbkv::clear_error() { g_err[0] = 0; }

namespace {

int fail_hip(hipError_t e, const char *what) {
    return fail(PBKV_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

int elt_bytes(int dtype) { return dtype == PBKV_BF16 ? 2 : 4; }

// Shape checks that need no device.  `need_heads` = the call uses the query-head count.
int check_shape(const pbkv_shape *s, bool need_heads) {
    if (!s) return fail(PBKV_ERR_NULL, "shape is NULL");
    if (s->dtype != PBKV_BF16 && s->dtype != PBKV_F32) return fail(PBKV_ERR_DTYPE, "unknown dtype %d", s->dtype);
    if (s->page_size != 16) return fail(PBKV_ERR_SHAPE, "page_size %d unsupported (16)", s->page_size);
    if (s->head_dim != 64 && s->head_dim != 128)
        return fail(PBKV_ERR_SHAPE, "head_dim %d unsupported (64, 128)", s->head_dim);
    if (s->num_kv_heads <= 0) return fail(PBKV_ERR_SHAPE, "num_kv_heads %d", s->num_kv_heads);
    if (s->num_pages <= 0) return fail(PBKV_ERR_SHAPE, "num_pages %d", s->num_pages);
    // the attention kernel addresses pool pages by 32-bit offsets in units of 256 bytes
    if ((int64_t)s->num_pages * 2 * s->num_kv_heads * s->page_size * s->head_dim * elt_bytes(s->dtype) >= ((int64_t)1 << 40))
        return fail(PBKV_ERR_LIMIT, "pool of %d pages is 1 TiB or more", s->num_pages);
    if (need_heads) {
        if (s->num_q_heads <= 0 || s->num_q_heads % s->num_kv_heads != 0)
            return fail(PBKV_ERR_SHAPE, "num_q_heads %d is not a multiple of num_kv_heads %d",
                        s->num_q_heads, s->num_kv_heads);
        const int G = s->num_q_heads / s->num_kv_heads;
        if (s->dtype == PBKV_BF16 && !(G == 1 || G == 2 || G == 4 || G == 8 || G == 16))
            return fail(PBKV_ERR_SHAPE, "query/KV head ratio %d unsupported for bf16 (1,2,4,8,16)", G);
    }
    if (s->batch < 0 || s->max_pages_per_req < 0) return fail(PBKV_ERR_SHAPE, "negative batch or table width");
    return PBKV_OK;
}

int check_lens(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens, int64_t *total) {
    int64_t N = 0;
    for (int r = 0; r < s->batch; r++) {
        const int64_t p = prefix_lens[r], n = new_lens[r];
        if (p < 0 || n < 0) return fail(PBKV_ERR_RANGE, "request %d: negative length (%lld, %lld)", r, (long long)p, (long long)n);
        if (p + n > INT32_MAX - 4096) return fail(PBKV_ERR_RANGE, "request %d: sequence too long", r);
        const int64_t pages = n > 0 ? (p + n + s->page_size - 1) / s->page_size : (p + s->page_size - 1) / s->page_size;
        if (n > 0 && pages > s->max_pages_per_req)
            return fail(PBKV_ERR_RANGE, "request %d needs %lld pages, block_table rows hold %d", r,
                        (long long)pages, s->max_pages_per_req);
        N += n;
    }
    *total = N;
    return PBKV_OK;
}

// The longest fp32 prefill call: MAX_F32_BLOCKS blocks of 64 suffix tokens, and rows (token, query head of a group) that
// 32-bit numbers count (past that, q alone is 512 GiB).
constexpr int64_t MAX_F32_BLOCKS = 131072;
int check_f32_length(const pbkv_shape *s, const int32_t *new_lens) {
    int64_t blocks = 0;
    const int64_t G = s->num_q_heads / s->num_kv_heads;
    for (int r = 0; r < s->batch; r++) {
        blocks += ((int64_t)new_lens[r] + 63) / 64;
        if (new_lens[r] * G > INT32_MAX - 4096) return fail(PBKV_ERR_LIMIT, "request %d: %d tokens of %d query heads per KV head", r, new_lens[r], (int)G);
    }
    if (blocks > MAX_F32_BLOCKS) return fail(PBKV_ERR_LIMIT, "%lld blocks of 64 new tokens, at most %lld", (long long)blocks, (long long)MAX_F32_BLOCKS);
    return PBKV_OK;
}

int check_aligned(const void *p, const char *name) {
    if (((uintptr_t)p & 15) != 0) return fail(PBKV_ERR_SHAPE, "%s is not 16-byte aligned", name);
    return PBKV_OK;
}

// Pointer kinds are asked of the runtime the first time the calling thread sees an address and
// remembered after that (a model passes the same buffers layer after layer, and the query costs
// about as much as a kernel launch).  The check catches a host pointer passed by mistake; it is no
// guard against a buffer that is freed and re-allocated as something else between calls.
enum PtrKind : uint8_t { KIND_NONE = 0, KIND_DEVICE = 1, KIND_PINNED = 2 };
struct PtrMemo {
    const void *ptr[32] = {};
    uint8_t kind[32] = {};
    int next = 0;
    bool has(const void *p, uint8_t k) const {
        for (int i = 0; i < 32; i++)
            if (ptr[i] == p && kind[i] == k) return true;
        return false;
    }
    void put(const void *p, uint8_t k) { ptr[next] = p; kind[next] = k; next = (next + 1) & 31; }
};
thread_local PtrMemo g_ptr_memo;

// The pointer must be something a kernel on the current device may dereference.
int check_device_ptr(const void *p, const char *name) {
    if (g_ptr_memo.has(p, KIND_DEVICE)) return PBKV_OK;
    hipPointerAttribute_t a;
    hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(PBKV_ERR_DEVICE, "%s: not a device pointer (%s)", name, hipGetErrorString(e));
    }
    if (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged)
        return fail(PBKV_ERR_DEVICE, "%s: expected device memory", name);
    g_ptr_memo.put(p, KIND_DEVICE);
    return PBKV_OK;
}

int check_pinned_ptr(const void *p, const char *name, const void **dev_view) {
    *dev_view = p;               // pinned memory shares one virtual address between host and device
    if (g_ptr_memo.has(p, KIND_PINNED)) return PBKV_OK;
    hipPointerAttribute_t a;
    hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(PBKV_ERR_DEVICE, "%s: not pinned host memory (%s)", name, hipGetErrorString(e));
    }
    if (a.type != hipMemoryTypeHost && a.type != hipMemoryTypeManaged)
        return fail(PBKV_ERR_DEVICE, "%s: expected pinned host memory", name);
    g_ptr_memo.put(p, KIND_PINNED);
    return PBKV_OK;
}

// ---- per-device state -----------------------------------------------------------------------
// (1) A ring of pinned, device-mapped descriptor memory.  Work lists are written here by the host
//     and read by the kernels through the mapped pointer (no copy in front of a kernel); a region
//     is reused only after the event recorded behind its kernel has fired.
// (2) Per stream, a small cache of work lists in device memory.  A launch that reads its list from
//     the ring also stores a copy there (every work-group writes back the descriptor it read), and
//     a later call on the same stream with the same shape and lengths -- the next layer of the same
//     batch -- launches straight from that copy: no list is built, nothing is copied, no event is
//     recorded, and no work-group reads over the host link.  Slots are only ever written and read
//     by kernels of one stream, so stream order is all the protection they need.
// (3) Per stream, the scratch buffer of the partial results (decode: context slices; attention: ranges of
//     KV tiles) and the counters that tell a decode work-group that it is the last of its request, for the
//     same reason: calls on different streams never share one.
struct Ring {
    char *host = nullptr;
    char *dev = nullptr;
    size_t cap = 0, head = 0;
    struct Pending { hipEvent_t ev; size_t begin, end; };
    std::deque<Pending> pending;
    std::vector<hipEvent_t> spare;
};
constexpr size_t RING_BYTES = 8u << 20;
constexpr int MAX_DEVICES = 16;
constexpr int PLAN_SLOTS = 16;                  // cached work lists per stream
constexpr size_t PLAN_SLOT_BYTES = 160u << 10;  // longer lists are not cached (every cut launch's list fits: MAX_CUT_UNITS)
constexpr int MAX_STREAM_CACHES = 8;            // streams with a cache, per device
constexpr int64_t DECODE_ONE_KERNEL_WGS = 1024; // work-groups of a decode call that merges in one kernel (see DECODE_ONE_KERNEL_BYTES)
constexpr int DECODE_COUNTERS = DECODE_ONE_KERNEL_WGS;   // its (request, KV head) pairs: each has a work-group at least

enum PlanKind { PLAN_ATTN = 1, PLAN_APPEND = 2, PLAN_DECODE = 3 };
struct Plan {
    bool valid = false;
    int kind = 0, forced_waves = 0;
    pbkv_shape shape{};
    std::vector<int32_t> lens;   // the host arrays the list was cut from, back to back
    int32_t n_a = 0, n_b = 0;    // items (tiles, merges | runs | slices, pages per slice)
    int32_t n_c = 0;             // attention: work-groups per KV head, where the list names them
    int32_t waves = 0;           // decode: one kernel
    int32_t key_groups = 1, most_parts = 0;      // attention
    int64_t aux = 0;             // bytes of scratch the launch needs
    uint64_t stamp = 0;
};
struct StreamCache {
    bool used = false;
    hipStream_t stream = nullptr;
    uint64_t thread = 0;         // of a per-thread stream, whose handle is the same on every thread; 0 for all others
    uint64_t stamp = 0;
    char *arena = nullptr;       // PLAN_SLOTS * PLAN_SLOT_BYTES of device memory
    Plan plans[PLAN_SLOTS];
    float *scratch = nullptr;    // partial results
    size_t scratch_cap = 0;
    uint32_t *counters = nullptr;   // DECODE_COUNTERS words, zero between decode launches
};
struct DevState {
    std::mutex mu;               // held from the first look at this state until the kernels are enqueued
    Ring ring;
    StreamCache sc[MAX_STREAM_CACHES];
    uint64_t clock = 0;
};
DevState g_dev[MAX_DEVICES];

int device_state(DevState **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(PBKV_ERR_DEVICE, "device index %d unsupported", dev);
    *out = &g_dev[dev];
    return PBKV_OK;
}

struct Lease { Ring *ring; size_t begin, end; char *host; char *dev; };

int ring_acquire(DevState &ds, size_t bytes, Lease *out) {
    Ring &r = ds.ring;
    hipError_t e;
    if (!r.host) {
        void *h = nullptr, *d = nullptr;
        e = hipHostMalloc(&h, RING_BYTES, hipHostMallocMapped);
        if (e != hipSuccess) return fail_hip(e, "hipHostMalloc(descriptor ring)");
        e = hipHostGetDevicePointer(&d, h, 0);
        if (e != hipSuccess) return fail_hip(e, "hipHostGetDevicePointer");
        r.host = (char *)h;
        r.dev = (char *)d;
        r.cap = RING_BYTES;
    }
    bytes = (bytes + 255) & ~(size_t)255;
    if (bytes > r.cap / 2) return fail(PBKV_ERR_LIMIT, "work list of %zu bytes exceeds the descriptor ring", bytes);
    if (r.head + bytes > r.cap) r.head = 0;
    const size_t b = r.head, en = r.head + bytes;
    // retire finished regions, wait for unfinished ones that overlap the new region
    for (auto it = r.pending.begin(); it != r.pending.end();) {
        const bool overlap = it->begin < en && it->end > b;
        hipError_t q = overlap ? hipEventSynchronize(it->ev) : hipEventQuery(it->ev);
        if (q == hipSuccess) {
            r.spare.push_back(it->ev);
            it = r.pending.erase(it);
        } else if (q == hipErrorNotReady) {
            ++it;
        } else {
            return fail_hip(q, "descriptor ring event");
        }
    }
    r.head = en;
    *out = Lease{&r, b, en, r.host + b, r.dev + b};
    return PBKV_OK;
}

// Record "the kernels reading this lease are enqueued" on the stream.
int ring_release(const Lease &l, hipStream_t s) {
    Ring &r = *l.ring;
    hipEvent_t ev;
    if (!r.spare.empty()) {
        ev = r.spare.back();
        r.spare.pop_back();
    } else {
        hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e != hipSuccess) return fail_hip(e, "hipEventCreate");
    }
    hipError_t e = hipEventRecord(ev, s);
    if (e != hipSuccess) return fail_hip(e, "hipEventRecord");
    r.pending.push_back({ev, l.begin, l.end});
    return PBKV_OK;
}

// A number for the calling thread that no other thread ever has.
uint64_t this_thread() {
    static std::atomic<uint64_t> threads{0};
    thread_local const uint64_t mine = ++threads;
    return mine;
}

// The cache of the stream; a stream seen for the first time takes an unused entry, or the entry
// used longest ago (its slots may still be read by that other stream's kernels: the device is
// drained first -- this only happens to callers that rotate over more than MAX_STREAM_CACHES streams).
// Callers that can do without (fp32 prefill) get null where there is no unused entry, or no memory for one: they would
// otherwise wait where they never had to.
int stream_cache(DevState &ds, hipStream_t st, bool must, StreamCache **out) {
    StreamCache *pick = nullptr;
    const uint64_t thread = st == hipStreamPerThread ? this_thread() : 0;
    for (auto &c : ds.sc) {
        if (c.used && c.stream == st && c.thread == thread) {
            c.stamp = ++ds.clock;
            *out = &c;
            return PBKV_OK;
        }
        if (!pick || (pick->used && (!c.used || c.stamp < pick->stamp))) pick = &c;
    }
    hipError_t e;
    *out = nullptr;
    if (pick->used && !must) return PBKV_OK;
    if (pick->used) {
        if ((e = hipDeviceSynchronize()) != hipSuccess) return fail_hip(e, "hipDeviceSynchronize");
        for (auto &pl : pick->plans) pl.valid = false;
    }
    if (!pick->arena) {
        void *m = nullptr;
        if ((e = hipMalloc(&m, PLAN_SLOTS * PLAN_SLOT_BYTES)) != hipSuccess) {
            (void)hipGetLastError();
            return must ? fail_hip(e, "hipMalloc(work-list cache)") : PBKV_OK;
        }
        pick->arena = (char *)m;
    }
    pick->used = true;
    pick->stream = st;
    pick->thread = thread;
    pick->stamp = ++ds.clock;
    *out = pick;
    return PBKV_OK;
}

bool same_shape(const pbkv_shape &a, const pbkv_shape &b) {
    return a.batch == b.batch && a.num_q_heads == b.num_q_heads && a.num_kv_heads == b.num_kv_heads &&
           a.head_dim == b.head_dim && a.page_size == b.page_size && a.dtype == b.dtype;
}

// The cached list for (kind, shape, lengths), or null.  `b` may be null (one array only).
Plan *find_plan(DevState &ds, StreamCache &c, int kind, const pbkv_shape *s, int forced_waves, const int32_t *a,
                const int32_t *b, char **dev) {
    const size_t n = (size_t)s->batch;
    for (int i = 0; i < PLAN_SLOTS; i++) {
        Plan &pl = c.plans[i];
        if (!pl.valid || pl.kind != kind || pl.forced_waves != forced_waves || !same_shape(pl.shape, *s)) continue;
        if (pl.lens.size() != (b ? 2 * n : n)) continue;
        if (memcmp(pl.lens.data(), a, n * sizeof(int32_t)) != 0) continue;
        if (b && memcmp(pl.lens.data() + n, b, n * sizeof(int32_t)) != 0) continue;
        pl.stamp = ++ds.clock;
        *dev = c.arena + (size_t)i * PLAN_SLOT_BYTES;
        return &pl;
    }
    return nullptr;
}

// The slot a new list goes to (least recently used); the caller fills in counts and marks it valid.
Plan *new_plan(DevState &ds, StreamCache &c, int kind, const pbkv_shape *s, int forced_waves, const int32_t *a,
               const int32_t *b, char **dev) {
    int pick = 0;
    for (int i = 0; i < PLAN_SLOTS; i++) {
        if (!c.plans[i].valid) { pick = i; break; }
        if (c.plans[i].stamp < c.plans[pick].stamp) pick = i;
    }
    Plan &pl = c.plans[pick];
    const size_t n = (size_t)s->batch;
    pl.valid = false;
    pl.kind = kind;
    pl.forced_waves = forced_waves;
    pl.shape = *s;
    pl.lens.assign(a, a + n);
    if (b) pl.lens.insert(pl.lens.end(), b, b + n);
    pl.stamp = ++ds.clock;
    *dev = c.arena + (size_t)pick * PLAN_SLOT_BYTES;
    return &pl;
}

// Scratch for the partial results of the decode and attention kernels on this stream, kept until the process ends.
// It grows by half as much again as a call asks for, so that growing calls re-allocate rarely, but attention never takes it past
// the most that one of its launches can ask for.  A buffer that is replaced is given back once the stream, whose kernels
// are its only readers, has run dry.  Where there is no memory for a larger one, the old one stays for the calls that fit it,
// unless the caller cannot go on without (`must`: decode; an attention launch runs whole).
constexpr int64_t MAX_CUT_UNITS = 2560;         // work-groups of an attention launch that leaves partial results
constexpr size_t CUT_SCRATCH_BYTES = (size_t)MAX_CUT_UNITS * 128 * (128 + 2) * sizeof(float);   // 162.5 MiB, at d = 128

int stream_scratch(StreamCache &c, size_t bytes, bool must, float **out) {
    if (c.scratch_cap < bytes) {
        auto give_back = [&]() {
            hipError_t e = c.scratch ? hipStreamSynchronize(c.stream) : hipSuccess;
            if (e != hipSuccess) return e;
            if (c.scratch) (void)hipFree(c.scratch);
            c.scratch = nullptr;
            c.scratch_cap = 0;
            return hipSuccess;
        };
        size_t cap = std::max({bytes, std::min(bytes + bytes / 2, CUT_SCRATCH_BYTES), (size_t)8 << 20});
        void *ptr = nullptr;
        hipError_t e = hipMalloc(&ptr, cap), g = hipSuccess;
        if (e != hipSuccess) e = hipMalloc(&ptr, cap = bytes);
        if (e == hipSuccess || must) g = give_back();
        if (e != hipSuccess && must && g == hipSuccess) e = hipMalloc(&ptr, cap);
        if (cap == bytes) (void)hipGetLastError();      // (an attempt may have failed: no error of a later call)
        if (g != hipSuccess) {
            if (e == hipSuccess) (void)hipFree(ptr);
            return fail_hip(g, "hipStreamSynchronize");
        }
        if (e != hipSuccess) return fail_hip(e, "hipMalloc (scratch of the partial results)");
        c.scratch = (float *)ptr;
        c.scratch_cap = cap;
    }
    *out = c.scratch;
    return PBKV_OK;
}

// The counters of this stream, or null where there is no memory for them: a second kernel merges then, with the same bits.
void decode_counters(StreamCache &c, uint32_t **out) {
    if (!c.counters) {
        void *ptr = nullptr;
        if (hipMalloc(&ptr, DECODE_COUNTERS * sizeof(uint32_t)) != hipSuccess) {
            (void)hipGetLastError();
            ptr = nullptr;
        } else if (pbkv::launch_clear_words((uint32_t *)ptr, DECODE_COUNTERS, c.stream) != hipSuccess) {
            (void)hipFree(ptr);
            ptr = nullptr;
        }
        c.counters = (uint32_t *)ptr;
    }
    *out = c.counters;
}

// Work lists live in library-owned memory that later calls reuse, so a captured graph would
// replay against lists that are gone: the entry points that use them refuse a capturing stream.
int check_not_capturing(hipStream_t st, const char *who) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(st, &status);
    if (e != hipSuccess) return fail_hip(e, "hipStreamIsCapturing");
    if (status != hipStreamCaptureStatusNone)
        return fail(PBKV_ERR_DEVICE, "%s: the stream is being captured into a graph; this call cannot be replayed", who);
    return PBKV_OK;
}

constexpr int MI355X_CUS = 256;

// How the attention kernels number the rows and keys of a request.
//   bf16: a row is a suffix token; KV tiles of 64 keys, the prefix's first (the last one may be partial),
//         then the suffix's
//   fp32: a row is a suffix token's query head of the group; tiles of 32 keys through prefix and suffix
struct Blocks {
    int T;              // rows per block
    int rows_per_tok;
    bool f32;
    int G, wg_rows;     // bf16: query heads per KV head; (token, query head) rows of a work-group
    int64_t rows(int64_t n) const { return n * rows_per_tok; }
    int64_t count(int64_t n) const { return (rows(n) + T - 1) / T; }
    // work-groups per KV head that hold rows of n suffix tokens (a block is a whole number of work-groups)
    int64_t wgs(int64_t n) const { return f32 ? count(n) : (n * G + wg_rows - 1) / wg_rows; }
    // KV tiles that the first `tok` suffix tokens see
    int64_t tiles(int64_t p, int64_t tok) const {
        if (f32) return (p + tok + pbkv::F32_KEYS - 1) / pbkv::F32_KEYS;
        return (p + pbkv::KV_TILE - 1) / pbkv::KV_TILE + (tok + pbkv::KV_TILE - 1) / pbkv::KV_TILE;
    }
    // the last tile whose first key every row of block k sees: the one that holds the block's first token
    int64_t last_start(int64_t p, int64_t k) const { return tiles(p, k * T / rows_per_tok + 1) - 1; }
};

// Work list of the attention kernels: one tile per block of rows of a request; `index` keeps
// the tile's index in request order.  Order: requests by descending length (prefix + suffix), and
// inside a request its token blocks from the last (most visible keys) to the first.  Long work goes
// first, so the launch ends on short work-groups, and the token blocks of one request -- which all
// stream the same K/V pages -- are handed out together: with KV head = work-group index mod H_kv
// they land on one XCD, run side by side and find each other's pages in its L2.  (Sorting the
// tiles of all requests by length alone interleaves requests of similar length; each then streams
// its prefix once per generation of its tiles: measured 2.5 - 3.6 times the compulsory HBM reads
// on the long-history and mixed batches.)
// A tile becomes wgs_per_tile consecutive work-groups; resident_pairs_wgs > 0 names the number of
// work-groups the chip holds at once when it holds two per CU (see below), 0 switches that case off.
// max_kt > 0 deals a token block's KV tiles out to units of at most that many, with one entry of *ranges per tile and one of
// *merges per block that was cut (see choose_cut and choose_cut_f32); both stay empty otherwise.  Slots of partial results are counted
// by the work-groups that hold rows, block by block, as choose_cut counts them: its limit is that of the scratch, too (with
// as many slots per part as the longest request's blocks have work-groups, 560 requests of one new token beside one of 33 at
// 16/1 heads of 128 took 462 MiB for what are 128).
int build_tiles(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens, const Blocks &bl,
                std::vector<pbkv::TileDesc> *out, int wgs_per_tile = 1, int resident_pairs_wgs = 0,
                int max_kt = 0, std::vector<pbkv::RangeDesc> *ranges_out = nullptr, std::vector<pbkv::MergeDesc> *merges = nullptr,
                int64_t *n_slots = nullptr) {
    std::vector<pbkv::TileDesc> &tiles = *out;
    tiles.clear();
    if (ranges_out) ranges_out->clear();
    if (merges) merges->clear();
    int32_t part = 0, slot = 0;
    thread_local std::vector<int32_t> order;
    thread_local std::vector<int64_t> row0, idx0;
    order.resize((size_t)s->batch);
    row0.resize((size_t)s->batch);
    idx0.resize((size_t)s->batch);
    int64_t rows = 0, idx = 0;
    for (int r = 0; r < s->batch; r++) {
        order[r] = r;
        row0[r] = rows;
        idx0[r] = idx;
        rows += new_lens[r];
        idx += bl.count(new_lens[r]);
    }
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return (int64_t)prefix_lens[a] + new_lens[a] > (int64_t)prefix_lens[b] + new_lens[b];
    });
    for (int32_t r : order) {
        const int32_t p = prefix_lens[r], n = new_lens[r];
        const int32_t T = bl.T, nb = (int32_t)bl.count(n), nt_max = (int32_t)bl.tiles(p, n);
        if (max_kt <= 0 || nt_max <= max_kt) {
            for (int32_t k = nb - 1; k >= 0; k--) {
                tiles.push_back(pbkv::TileDesc{r, k * T, p, n, row0[r], idx0[r] + k});
                if (max_kt > 0) ranges_out->push_back(pbkv::RangeDesc{-1, 0, INT32_MAX, 0});
            }
            continue;
        }
        // the same ranges for every token block of the request, range by range, so that the blocks that read
        // a range run side by side.  A range starts at a tile whose first key every row of the block sees: a bf16
        // work-group may hold the block's first rows alone, and takes at least one tile of its range.  (The fp32
        // kernel, whose work-group is the whole block, shares the rule without need for it.)
        const int32_t ranges = (nt_max + max_kt - 1) / max_kt, step = (nt_max + ranges - 1) / ranges;
        thread_local std::vector<int32_t> part0, slot0;
        part0.resize((size_t)nb);
        slot0.resize((size_t)nb);
        auto splits_of = [&](int32_t k) { return bl.f32 ? 1 : (int32_t)bl.wgs(std::min(T, n - k * T)); };
        auto ranges_of = [&](int32_t k) { return 1 + (int32_t)bl.last_start(p, k) / step; };
        for (int32_t k = 0; k < nb; k++) {
            const int32_t m = ranges_of(k);
            part0[k] = part;
            slot0[k] = slot;
            if (m > 1) {
                merges->push_back(pbkv::MergeDesc{k * T, n, part, m, row0[r], slot, splits_of(k)});
                part += m;
                slot += m * splits_of(k);
            }
        }
        for (int32_t c = 0; c < ranges; c++)
            for (int32_t k = nb - 1; k >= 0; k--) {
                const int32_t m = ranges_of(k);
                if (c >= m) continue;
                tiles.push_back(pbkv::TileDesc{r, k * T, p, n, row0[r], idx0[r] + k});
                ranges_out->push_back(pbkv::RangeDesc{m > 1 ? part0[k] + c : -1, c * step, c + 1 < m ? (c + 1) * step : INT32_MAX, slot0[k] + c * splits_of(k)});
            }
    }
    if (n_slots) *n_slots = slot;
    // A launch whose work-groups are all resident at once, two per CU (the 4-wave shape on 256 CUs),
    // finishes when the CU with the most work does, and the dispatcher hands out one work-group per CU
    // before it starts on the second: the second half of the list is reversed, so that the CU holding
    // the longest work-group also gets the shortest (measured +2 % on the shared-prompt batch's
    // attention launch running alone; no difference with the append kernel beside it).
    const size_t n = tiles.size();
    if (resident_pairs_wgs > 0 && n * (size_t)wgs_per_tile > (size_t)resident_pairs_wgs / 2 &&
        n * (size_t)wgs_per_tile <= (size_t)resident_pairs_wgs)
        std::reverse(tiles.begin() + (resident_pairs_wgs / 2 + wgs_per_tile - 1) / wgs_per_tile, tiles.end());
    if (tiles.size() > (size_t)INT32_MAX / 64) return fail(PBKV_ERR_LIMIT, "too many tiles");
    return PBKV_OK;
}

// Work-groups of a launch whose blocks are cut into ranges of at most `len` tiles; the longest block and the
// tile steps of all of them.
int64_t count_units(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens, const Blocks &bl,
                    int64_t len, int64_t *longest, int64_t *steps) {
    int64_t units = 0;
    *longest = *steps = 0;
    for (int r = 0; r < s->batch; r++) {
        const int64_t n = bl.wgs(new_lens[r]) * s->num_kv_heads, nt = bl.tiles(prefix_lens[r], new_lens[r]);
        if (n == 0) continue;
        units += n * ((nt + len - 1) / len);
        *steps += n * nt;
        *longest = std::max(*longest, nt);
    }
    return units;
}

// What a launch comes to whose blocks are cut into ranges of at most `len` tiles as build_tiles cuts them.
struct CutSize {
    int64_t units = 0;          // work-groups
    int64_t groups = 0;         // 32-row groups in those of them that leave a partial result
    int64_t longest = 0;        // tile steps of the longest
};
CutSize cut_size(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens, const Blocks &bl, int64_t len) {
    CutSize c;
    for (int r = 0; r < s->batch; r++) {
        const int64_t p = prefix_lens[r], n = new_lens[r], nt_max = bl.tiles(p, n);
        const int64_t ranges = (nt_max + len - 1) / len, step = n > 0 ? (nt_max + ranges - 1) / ranges : 1;
        for (int64_t k = 0, nb = bl.count(n); k < nb; k++) {
            const int64_t per_tile = bl.wgs(std::min<int64_t>(bl.T, n - k * bl.T)) * s->num_kv_heads;
            const int64_t nt = bl.tiles(p, std::min((k + 1) * bl.T, bl.rows(n)) / bl.rows_per_tok), m = 1 + bl.last_start(p, k) / step;
            c.units += m * per_tile;
            if (m > 1) c.groups += m * ((std::min<int64_t>(bl.T, n - k * bl.T) * bl.G + 31) / 32) * s->num_kv_heads;
            c.longest = std::max(c.longest, m > 1 ? std::max(step, nt - (m - 1) * step) : nt);
        }
    }
    return c;
}

// Whether that pays, against launching the blocks whole in the 4-wave shape.  The second kernel, the partial results and
// a second prologue are weighed against the steps that the longest work-group is shorter by; the lines are those of 500
// drawn launches that were timed both ways (largest loss on the wrong side of a line 17 %, without the lines 51 %).
//   All work-groups on a CU of their own: the cost is 3 steps and one per 25 whole work-groups at d = 128, whose steps are
//   longer, 4 and one per 50 at d = 64.  us whole and cut: 13 requests of 6 tiles at 4/2 heads of 128 12.0 and
//   18.1; 5 of 5 tiles 10.5 and 15.1; one of 131 + 220 tokens at 8/2 16.2 and 12.3; 3 of 290 + 290 at 16/1 heads of 64 10.3 and 13.5.
//   More work-groups than CUs: a step of two that share a CU takes a quarter longer, and the partial results pass through
//   memory at one step per 25 (d = 64, half their size: per 30): 3 of 20 tiles at 16/2 heads of 128 (408 work-groups) 29.2 and 39.3, 6 of
//   17 + 1281 tokens at 4/2 29.6 and 38.7, one of 5086 + 718 at 32/8 93.9 and 89.8; 3 of 1836 + 120 .. 633 at 16/2 heads of 64 34.2 and 28.3.
//   Partial results are counted by their 32-row groups that hold rows (16 KiB each at d = 128).
//   Against two key groups (below) the whole launch counts as 0.82 of its steps at d = 128, 0.85 at 64.
bool ranges_pay(int head_dim, const CutSize &whole, const CutSize &cut, bool two_groups) {
    const int64_t longest = !two_groups ? whole.longest : head_dim == 128 ? whole.longest * 82 / 100 : whole.longest * 85 / 100;
    if (cut.units <= MI355X_CUS)
        return head_dim == 128 ? 25 * (longest - cut.longest - 3) > whole.units : 50 * (longest - cut.longest - 4) > whole.units;
    const int per_step = head_dim == 128 ? 25 : 30;
    return per_step * (4 * longest - 5 * cut.longest) > cut.groups;
}

// A whole 4-wave launch whose work-groups each have a CU to themselves, and their first tile steps behind them: a second key group
// per work-group uses the other half of the CU.  us with one group and two, by steps of the longest work-group, means of
// 250 drawn launches of up to 256 work-groups: at d = 128 2 .. 4 steps +5 %, 5 or 6 +1 %, 7 .. 9 -4 %, 10 .. 14 -7 %,
// 15 .. 24 -11 %, beyond 100 -20 %; at d = 64 5 or 6 -1 %, 7 .. 9 -5 %, 15 .. 24 -17 %, beyond 100 -28 %.  With more work-groups
// than CUs it loses 10 .. 50 %: a second work-group on the CU overlaps its first and last steps with the other's arithmetic.
constexpr int64_t TWO_GROUPS_STEPS = 8;

// The same for a cut launch: 32 parts at most leave CUs idle where few KV heads have long contexts, and the ranges are long then. us, one group
// and two: 32000 + 25 tokens at 16/2 heads of 64 (128 work-groups of 16 steps) 20.1 and 17.9, + 3 (64 of 16) 17.6 and 15.6, + 62 (256 of 16)
// 21.6 and 20.6; 32000 + 12 at 32/2 heads of 128 (128 of 16) 25.7 and 24.3; 16000 + 25 at 16/2 of 64 (128 of 8) 14.4 and 13.9.  With shorter
// ranges the meeting costs more (8000 + 25 at 16/2 of 64, ranges of 4: 12.4 and 12.7), and where every CU streams from HBM there
// is nothing to gain (12001 + 37 at 32/8 of 128 20.6 and 21.0, 32000 + 30 29.3 and 30.6).
bool two_groups_in_ranges(int head_dim, int64_t units, int64_t steps) {
    return (units <= MI355X_CUS / 2 && steps >= (head_dim == 128 ? 12 : 8)) || (head_dim == 64 && units <= MI355X_CUS && steps >= 12);
}

// How a bf16 attention launch is cut: the work-group shape, and the most KV tiles of a unit (0: a unit
// takes all tiles of its token block).  Dealing a block's keys out to several units costs a second
// kernel (4 us) and a store and a read of 64 KiB per unit, so it is done where the launch would otherwise
// leave CUs idle, with the 4-wave shape.  GPU times per call, 32/8 heads of 128, and of 64 in brackets:
//   fewer token blocks than the chip holds work-groups (prefix + new tokens: uncut, in the shape the launch would have, -> cut):
//     12001 + 37 247 -> 24 us [168 -> 18], 32768 + 1 646 -> 34, 32768 + 512 659 -> 254 [453 -> 154], 8000 + 200 171 -> 42 [116 -> 25],
//     500 + 32 15.2 -> 9.9 [11.5 -> 8.8].  With ranges of up to 20 tiles one work-group per CU is the better aim (12001 + 37: 22 us in
//     ranges of 12, 25 of 6 [16, 18]; 8 x (2000 + 64): 33 of 20 or more, 41 of 6 [23, 26]), with longer ones two (32768 +
//     512: 254 in ranges of 160, 278 of 260 [150, 182]).  Ranges of fewer than 4 tiles gain where they leave no more
//     parts than the merge takes in one trip (whole -> as short as that allows: 300 + 8 11.2 -> 8.9 us, 700 + 10 16.4 -> 9.2, 200 + 64
//     12.2 -> 9.7); past it they do not (2000 + 20 at 8/2 heads of 64, 33 tiles: 10.5 in ranges of 4, 12.0 of 1).  No block is cut into
//     more than 32 parts, the merge's second step (14640 + 37 at 8/2 heads of 64: 17.6 us in 58 parts, 13.9 in 29; 20000 + 6 24.4 in
//     40, 20.4 in 32), and a range is not shorter than a step's 0.9 us [0.6] is worth against 5 us [3.3] per 1000 of the 32-row
//     groups of partial results: sqrt(groups x tiles / 180) tiles (3 x (599 .. 1142 + 39) at 32/2: 18.1 in ranges of 2, 15.0 of 4).
//   64-row units that do not fill their rounds over the CUs (264 units of 533 steps on 256 CUs: 1556 -> 1128 us [990 -> 667]; 288
//     of 268: 774 -> 623 [493 -> 365]; 144 of 268: 359 -> 320 [247 -> 190]): cut when the 64-row form's makespan (of the work-groups that
//     hold rows) exceeds 1.35 [1.2] times the even share of its 4-wave units (of which a 64-row unit of up to 128 rows is one, and
//     so half as long) over the 512 places.  230 drawn launches timed whole and cut: below 1.2 from -12 to +18 % by the cut, at d = 64 above
//     it -3 .. -51 %, at d = 128 above 1.35 -4 .. -31 %.  The 4-wave units of a request's one or two 64-row units, and all of one KV
//     head, do not meet in one XCD's L2 unless the KV heads are a multiple of its eight: its keys come more often from HBM, and at
//     d = 128 the line is 1.6: us, n x (12800 + 16) tokens at 16/1, whole and cut, 520 [1.48 times] 985, 1053; 340 [1.51] 655, 661; 260 [1.97] 629, 563; 98 x
//     (9867 + 31) at 32/2 [1.31] +16 %, 87 x (12584 + 12) at 64/4 [1.47] +11 %; and 520 x (12800 + 1) at 16/1 [2.96] 938, 638.  Four ranges' worth of work per place, at least 48 tiles each: 264 units
//     of 533 steps take 1127 us with ranges of 160 tiles, 1151 with ranges of 260 [665, 688].
struct AttnCut { int waves, max_kt, key_groups = 1; };

Blocks blocks_bf16(const pbkv_shape *s, int waves) {
    const int G = s->num_q_heads / s->num_kv_heads;
    return Blocks{pbkv::attn_bf16_tile_tokens(s->head_dim, G, waves), 1, false, G, waves == 4 ? 128 : 256};
}

// The work-group shape of a launch that is not cut.  The 4-wave form reads the Q rows of a wave at 32-bit offsets from its
// first token; where 32 / G tokens are 2 GiB or more (262144 heads of 128 at G = 1) the 8-wave form, which addresses every row in
// 64 bits, takes its place.  Offsets from two points per wave instead cost 0.4 % over 16 launches of 5 .. 110 us.  (A launch that is cut has fewer
// than 1024 work-groups, so fewer heads than that by far.)
int whole_waves(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens) {
    const int waves = pbkv::attn_bf16_waves(prefix_lens, new_lens, s->batch);
    const int64_t G = s->num_q_heads / s->num_kv_heads, span = (32 / G) * s->num_q_heads * s->head_dim * 2;
    return waves == 4 && span > INT32_MAX ? 8 : waves;
}

AttnCut choose_cut(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens) {
    const int waves = whole_waves(s, prefix_lens, new_lens);
    if (pbkv::attn_bf16_forced_waves()) return {waves, 0};
    constexpr int64_t SLOTS = 2 * MI355X_CUS;   // work-groups of the 4-wave shape that run at once
    // work-groups and tile steps of the launch when every token block is cut into ranges of `len` tiles
    int64_t longest = 0, steps = 0;
    const Blocks b4 = blocks_bf16(s, 4);
    auto units_at = [&](const Blocks &bl, int64_t len) { return count_units(s, prefix_lens, new_lens, bl, len, &longest, &steps); };
    const int64_t units4 = units_at(b4, INT32_MAX), steps4 = steps;
    if (units4 == 0) return {waves, 0};
    if (units4 < SLOTS) {
        int64_t groups = 0;                      // 32-row groups of the launch
        for (int r = 0; r < s->batch; r++) groups += ((int64_t)new_lens[r] * b4.G + 31) / 32 * s->num_kv_heads;
        int64_t shortest = std::max<int64_t>(std::min<int64_t>(4, (longest + pbkv::MERGE_AHEAD - 1) / pbkv::MERGE_AHEAD),
                                             (longest + 2 * pbkv::MERGE_AHEAD - 1) / (2 * pbkv::MERGE_AHEAD));
        while (180 * (shortest + 1) * (shortest + 1) <= groups * longest) shortest++;
        auto length_for = [&](int64_t wgs) {     // smallest length with which no more than `wgs` units exist
            int64_t len = std::max<int64_t>((steps4 + wgs - 1) / wgs, shortest);
            while (len < longest && units_at(b4, len) > wgs) len += std::max<int64_t>(1, len / 8);
            return len;
        };
        int64_t len = length_for(SLOTS / 2);
        if (len > 20) len = length_for(SLOTS);
        const bool two_groups = units4 <= MI355X_CUS && longest >= TWO_GROUPS_STEPS;
        // (a launch that would otherwise run in the 64-row form gains from any cut: that form has half the work-groups)
        if (len + 4 <= longest &&
            (waves == 64 || ranges_pay(s->head_dim, cut_size(s, prefix_lens, new_lens, b4, INT32_MAX),
                                       cut_size(s, prefix_lens, new_lens, b4, len), two_groups)))
            return {4, (int)len, two_groups_in_ranges(s->head_dim, units_at(b4, len), len) ? 2 : 1};
        if (waves == 4 && two_groups) return {4, 0, 2};
    }
    if (waves != 64) return {waves, 0};
    // list scheduling of the 64-row units, those that hold rows, on a CU each
    const Blocks b64 = blocks_bf16(s, 64);
    const int64_t units64 = units_at(b64, INT32_MAX);
    if (units64 > 4 * MI355X_CUS) return {waves, 0};
    thread_local std::vector<int64_t> busy;
    thread_local std::vector<int32_t> lens;
    busy.assign(MI355X_CUS, 0);                  // a heap, the least busy first
    lens.clear();
    int64_t total = 0, total4 = 0, makespan = 0, lone = 0;      // tile steps
    const int32_t wg_tok = b64.wg_rows / b64.G, wg_tok4 = b4.wg_rows / b4.G;
    for (int r = 0; r < s->batch; r++) {
        for (int32_t t0 = 0; t0 < new_lens[r]; t0 += wg_tok) {
            lens.push_back((int32_t)b64.tiles(prefix_lens[r], std::min(t0 + wg_tok, new_lens[r])));
            if (2 * new_lens[r] > wg_tok && new_lens[r] <= 2 * (int64_t)wg_tok) lone += (int64_t)lens.back() * s->num_kv_heads;
        }
        for (int32_t t0 = 0; t0 < new_lens[r]; t0 += wg_tok4) total4 += b4.tiles(prefix_lens[r], std::min(t0 + wg_tok4, new_lens[r])) * s->num_kv_heads;
    }
    std::sort(lens.begin(), lens.end(), [](int32_t a, int32_t b) { return a > b; });
    for (int32_t n : lens)
        for (int h = 0; h < s->num_kv_heads; h++) {
            std::pop_heap(busy.begin(), busy.end(), std::greater<int64_t>());
            makespan = std::max(makespan, busy.back() += n);
            std::push_heap(busy.begin(), busy.end(), std::greater<int64_t>());
            total += n;
        }
    const bool spread = s->num_kv_heads == 1 || (s->num_kv_heads % 8 != 0 && 2 * lone > total);
    const int64_t line = s->head_dim == 64 ? 120 : spread ? 160 : 135;
    if (100 * makespan * SLOTS <= line * total4) return {waves, 0};
    const int64_t len = std::max<int64_t>(48, (steps4 + 4 * SLOTS - 1) / (4 * SLOTS));
    if (units_at(b4, len) > MAX_CUT_UNITS) return {waves, 0};
    return {4, (int)len};
}

// The fp32 launch: most KV tiles of a unit, 0 for all.  A tile step of a work-group keeps all four matrix
// pipes of a CU busy (3.9 us at d = 128, half at 64), so one work-group per CU is the aim and a launch that
// has that many is left whole.  The second kernel costs about as much as one or two steps.  us per call,
// whole -> cut (2/1 heads of 64): 256 + 64 tokens 32.4 -> 12.5, 2048 + 256 207 -> 19; (8/2 heads of 128): 50 + 50
// 23.8 -> 17.0 (ranges of one tile, the shortest context that is cut has three), 2048 + 256 358 -> 41, four of
// these 368 -> 106 (ranges of 20 tiles; of 8 to 12: 121 to 130).
int choose_cut_f32(const pbkv_shape *s, const int32_t *prefix_lens, const int32_t *new_lens, const Blocks &bl) {
    int64_t longest = 0, steps = 0;
    auto units_at = [&](int64_t len) { return count_units(s, prefix_lens, new_lens, bl, len, &longest, &steps); };
    const int64_t units = units_at(INT32_MAX);
    if (units >= MI355X_CUS || pbkv::attn_bf16_forced_waves()) return 0;      // (a forced shape: results that no batch changes)
    int64_t len = std::max<int64_t>((steps + MI355X_CUS - 1) / MI355X_CUS, 1);
    while (len < longest && units_at(len) > MI355X_CUS) len += std::max<int64_t>(1, len / 8);
    return len + 2 <= longest ? (int)len : 0;
}

thread_local std::vector<pbkv::TileDesc> tl_tiles;
thread_local std::vector<pbkv::RangeDesc> tl_ranges;
thread_local std::vector<pbkv::MergeDesc> tl_merges;
thread_local std::vector<uint32_t> tl_units;
thread_local std::vector<pbkv::AppendDesc> tl_runs;
thread_local std::vector<pbkv::DecodeReq> tl_reqs;
thread_local std::vector<uint8_t> tl_seen;
thread_local std::vector<int32_t> tl_ids;

}  // namespace

extern "C" {

const char *pbkv_last_error(void) { return g_err; }

const char *pbkv_version(void) { return "pbkv 0.2 gfx950"; }

int64_t pbkv_page_bytes(const pbkv_shape *s) {
    if (!s || check_shape(s, false) != PBKV_OK) return 0;
    return (int64_t)2 * s->num_kv_heads * s->page_size * s->head_dim * elt_bytes(s->dtype);
}

int pbkv_set_attn_waves(int waves) {
    g_err[0] = 0;
    if (waves != 0 && waves != 4 && waves != 8 && waves != 64) return fail(PBKV_ERR_SHAPE, "pbkv_set_attn_waves: %d (0, 4, 8 or 64)", waves);
    pbkv::attn_bf16_force_waves(waves);
    return PBKV_OK;
}

int pbkv_prefix_prefill(const pbkv_shape *s, const void *q, const void *k_new, const void *v_new,
                        const void *kv_pool, const int32_t *block_table, const int32_t *prefix_lens,
                        const int32_t *new_lens, void *out, void *stream) {
    g_err[0] = 0;
    int rc = check_shape(s, true);
    if (rc) return rc;
    if (s->batch == 0) return PBKV_OK;
    if (!q || !k_new || !v_new || !kv_pool || !block_table || !prefix_lens || !new_lens || !out)
        return fail(PBKV_ERR_NULL, "pbkv_prefix_prefill: NULL argument");
    int64_t N = 0;
    if ((rc = check_lens(s, prefix_lens, new_lens, &N))) return rc;
    if (N == 0) return PBKV_OK;
    if (s->dtype == PBKV_F32 && (rc = check_f32_length(s, new_lens))) return rc;
    if ((rc = check_aligned(q, "q")) || (rc = check_aligned(k_new, "k_new")) || (rc = check_aligned(v_new, "v_new")) ||
        (rc = check_aligned(kv_pool, "kv_pool")) || (rc = check_aligned(out, "out")))
        return rc;
    if ((rc = check_device_ptr(q, "q")) || (rc = check_device_ptr(k_new, "k_new")) ||
        (rc = check_device_ptr(v_new, "v_new")) || (rc = check_device_ptr(kv_pool, "kv_pool")) ||
        (rc = check_device_ptr(block_table, "block_table")) || (rc = check_device_ptr(out, "out")))
        return rc;

    hipStream_t st = (hipStream_t)stream;
    if ((rc = check_not_capturing(st, "pbkv_prefix_prefill"))) return rc;
    pbkv::AttnParams p;
    p.q = q; p.k_new = k_new; p.v_new = v_new; p.kv_pool = kv_pool; p.out = out;
    p.block_table = block_table;
    p.Hq = s->num_q_heads; p.Hkv = s->num_kv_heads;
    p.max_pages = s->max_pages_per_req; p.num_pages = s->num_pages;
    p.mirror = nullptr; p.ranges = nullptr; p.mirror_ranges = nullptr; p.key_groups = 1; p.most_parts = 0; p.splits = 1; p.row_groups = 0;
    p.units = nullptr; p.mirror_units = nullptr; p.n_units = 0;
    p.merges = nullptr; p.mirror_merges = nullptr; p.n_merges = 0; p.partial = nullptr;
    const bool bf16 = s->dtype == PBKV_BF16;
    const int G = s->num_q_heads / s->num_kv_heads;
    const int longest_new = *std::max_element(new_lens, new_lens + s->batch);
    // of the longest request's blocks, with the shape in p.waves
    auto set_rows = [&]() {
        if (!bf16) return;
        p.splits = pbkv::attn_bf16_splits(G, p.waves, longest_new);
        p.row_groups = std::min((int)(((int64_t)longest_new * G + 31) / 32), 4 * p.splits);
    };
    auto launch = [&]() {
        return bf16 ? pbkv::launch_attn_bf16(p, s->head_dim, st) : pbkv::launch_attn_f32(p, s->head_dim, st);
    };

    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    StreamCache *sc = nullptr;
    char *slot = nullptr;
    const int forced = pbkv::attn_bf16_forced_waves();
    if ((rc = stream_cache(*ds, st, bf16, &sc))) return rc;
    if (Plan *pl = !sc ? nullptr : find_plan(*ds, *sc, PLAN_ATTN, s, forced, prefix_lens, new_lens, &slot)) {
        p.tiles = (const pbkv::TileDesc *)slot;
        p.n_tiles = pl->n_a;
        p.waves = pl->waves;
        p.key_groups = pl->key_groups;
        p.most_parts = pl->most_parts;
        set_rows();
        p.n_merges = pl->n_b;
        if (p.n_merges > 0) {
            p.ranges = (const pbkv::RangeDesc *)(slot + (size_t)p.n_tiles * sizeof(pbkv::TileDesc));
            p.merges = (const pbkv::MergeDesc *)(p.ranges + p.n_tiles);
        }
        p.n_units = pl->n_c;
        if (p.n_units > 0) p.units = p.n_merges > 0 ? (const uint32_t *)(p.merges + p.n_merges) : (const uint32_t *)(p.tiles + p.n_tiles);
        if (pl->aux == 0 || stream_scratch(*sc, (size_t)pl->aux, false, &p.partial) == PBKV_OK) {
            g_err[0] = 0;
            hipError_t e = launch();
            return e == hipSuccess ? PBKV_OK : fail_hip(e, "attention launch");
        }
        pl->valid = false;                       // cut, and no memory for the partial results any more: rebuilt whole
        p.n_merges = 0;
        p.ranges = nullptr;
        p.merges = nullptr;
        p.units = nullptr;
    }

    AttnCut cut{0, 0};
    Blocks bl{pbkv::attn_f32_block_rows(), G, true, G, pbkv::attn_f32_block_rows()};
    int per_tile = s->num_kv_heads;              // work-groups per tile
    if (bf16) {
        cut = choose_cut(s, prefix_lens, new_lens);
        bl = blocks_bf16(s, cut.waves);
        per_tile = pbkv::attn_bf16_splits(G, cut.waves, longest_new) * s->num_kv_heads;
    } else if (sc) {
        cut.max_kt = choose_cut_f32(s, prefix_lens, new_lens, bl);
    }
    std::vector<pbkv::TileDesc> &tiles = tl_tiles;
    std::vector<pbkv::RangeDesc> &ranges = tl_ranges;
    std::vector<pbkv::MergeDesc> &merges = tl_merges;
    size_t scratch = 0;
    for (;;) {
        int64_t n_slots = 0;
        if ((rc = build_tiles(s, prefix_lens, new_lens, bl, &tiles, per_tile, cut.waves == 4 && cut.max_kt == 0 ? 2 * MI355X_CUS : 0,
                              cut.max_kt, &ranges, &merges, &n_slots)))
            return rc;
        const int64_t part_floats = bf16 ? pbkv::attn_bf16_partial_floats(s->head_dim) : pbkv::attn_f32_partial_floats(s->head_dim);
        scratch = (size_t)(n_slots * s->num_kv_heads * part_floats) * sizeof(float);
        if (scratch == 0 || stream_scratch(*sc, scratch, false, &p.partial) == PBKV_OK) break;
        // no memory for partial results: the launch runs whole, which needs none
        cut = AttnCut{bf16 ? whole_waves(s, prefix_lens, new_lens) : 0, 0};
        if (bf16) {
            bl = blocks_bf16(s, cut.waves);
            per_tile = pbkv::attn_bf16_splits(G, cut.waves, longest_new) * s->num_kv_heads;
        }
    }
    g_err[0] = 0;
    p.waves = cut.waves;
    p.key_groups = cut.key_groups;
    set_rows();
    p.most_parts = 0;
    for (const auto &m : merges) p.most_parts = std::max(p.most_parts, m.n_parts);
    if (merges.empty()) ranges.clear();           // no block has more tiles than a range: the launch is whole
    const size_t tb = tiles.size() * sizeof(pbkv::TileDesc), rb = ranges.size() * sizeof(pbkv::RangeDesc);
    const size_t mb = merges.size() * sizeof(pbkv::MergeDesc);
    // Tiles of fewer work-groups than the longest request's: the list names those that exist.  Work-groups go to the XCDs in turn, so the
    // places of those that do not would all be missing on the same XCDs, and the others take a second round: us with empty work-groups and
    // without: 2 x (13508 .. 54033 + 76) tokens at 16/2 heads of 64 48.6, 34.5; 12 x (29560 + 1 .. 15) at 64/4 of 128 248, 161; 27 x (8616 + 13 .. 105) at 32/2 302 (cut),
    // 247 (whole); 59 x (1098 + 3 .. 24) at 32/4 45.2, 37.2.  Where fewer than one in 32 is missing it costs more to read the list (0.4 us).
    std::vector<uint32_t> &units = tl_units;
    units.clear();
    if (bf16 && p.splits > 1)
        for (size_t t = 0; t < tiles.size() && tb + rb + mb + 4 * units.size() <= PLAN_SLOT_BYTES; t++)
            for (int k = 0, n = (int)bl.wgs(std::min(bl.T, tiles[t].new_len - tiles[t].tok0)); k < n; k++) units.push_back((uint32_t)(4 * t + k));
    const size_t ub = 4 * units.size();
    if (32 * units.size() > 31 * tiles.size() * p.splits || tb + rb + mb + ub > PLAN_SLOT_BYTES) units.clear();
    p.n_units = (int32_t)units.size();
    const size_t bytes = tb + rb + mb + 4 * units.size();

    Lease lease;
    // An fp32 block is 128 rows, however many query heads share a KV head, so an fp32 list may be longer than the ring takes at
    // a time: such a call goes out in several launches.  (So that no grid reaches 2^32 threads, too.)
    const size_t at_once = bf16 ? tiles.size() : std::min<size_t>(RING_BYTES / 4 / sizeof(pbkv::TileDesc), std::max<uint32_t>(1, UINT32_MAX / 256 / (uint32_t)s->num_kv_heads));
    if (tiles.size() > at_once) {
        for (size_t t0 = 0; t0 < tiles.size(); t0 += at_once) {
            p.n_tiles = (int32_t)std::min(at_once, tiles.size() - t0);
            if ((rc = ring_acquire(*ds, p.n_tiles * sizeof(pbkv::TileDesc), &lease))) return rc;
            memcpy(lease.host, tiles.data() + t0, p.n_tiles * sizeof(pbkv::TileDesc));
            p.tiles = (const pbkv::TileDesc *)lease.dev;
            hipError_t e = launch();
            if ((rc = ring_release(lease, st))) return rc;
            if (e != hipSuccess) return fail_hip(e, "attention launch");
        }
        return PBKV_OK;
    }
    if ((rc = ring_acquire(*ds, bytes, &lease))) return rc;
    memcpy(lease.host, tiles.data(), tb);
    memcpy(lease.host + tb, ranges.data(), rb);
    memcpy(lease.host + tb + rb, merges.data(), mb);
    memcpy(lease.host + tb + rb + mb, units.data(), bytes - tb - rb - mb);
    p.tiles = (const pbkv::TileDesc *)lease.dev;
    p.n_tiles = (int32_t)tiles.size();
    p.n_merges = (int32_t)merges.size();
    if (p.n_merges > 0) {
        p.ranges = (const pbkv::RangeDesc *)(lease.dev + tb);
        p.merges = (const pbkv::MergeDesc *)(lease.dev + tb + rb);
    }
    if (p.n_units > 0) p.units = (const uint32_t *)(lease.dev + tb + rb + mb);
    Plan *pl = nullptr;
    if (sc && bytes <= PLAN_SLOT_BYTES) {
        pl = new_plan(*ds, *sc, PLAN_ATTN, s, forced, prefix_lens, new_lens, &slot);
        pl->n_a = p.n_tiles;
        pl->n_b = p.n_merges;
        pl->n_c = p.n_units;
        pl->aux = (int64_t)scratch;
        pl->waves = cut.waves;
        pl->key_groups = cut.key_groups;
        pl->most_parts = p.most_parts;
        p.mirror = (pbkv::TileDesc *)slot;
        p.mirror_ranges = (pbkv::RangeDesc *)(slot + tb);
        p.mirror_merges = (pbkv::MergeDesc *)(slot + tb + rb);
        if (p.n_units > 0) p.mirror_units = (uint32_t *)(slot + tb + rb + mb);
    }
    hipError_t e = launch();
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "attention launch");
    if (pl) pl->valid = true;
    return rel;
}

int pbkv_gather_probe(const pbkv_shape *s, const void *k_new, const void *v_new, const void *kv_pool,
                      const int32_t *block_table, const int32_t *prefix_lens, const int32_t *new_lens,
                      uint32_t *unit_xor, int64_t unit_capacity, int64_t *n_units, int32_t *unit_tokens,
                      void *stream) {
    g_err[0] = 0;
    int rc = check_shape(s, true);
    if (rc) return rc;
    if (s->dtype != PBKV_BF16) return fail(PBKV_ERR_DTYPE, "pbkv_gather_probe: bf16 only");
    if (!n_units || !unit_tokens) return fail(PBKV_ERR_NULL, "pbkv_gather_probe: NULL argument");
    const int G = s->num_q_heads / s->num_kv_heads;
    *unit_tokens = pbkv::attn_bf16_tile_tokens(s->head_dim, G, 8);
    *n_units = 0;
    if (s->batch == 0) return PBKV_OK;
    if (!k_new || !v_new || !kv_pool || !block_table || !prefix_lens || !new_lens)
        return fail(PBKV_ERR_NULL, "pbkv_gather_probe: NULL argument");
    int64_t N = 0;
    if ((rc = check_lens(s, prefix_lens, new_lens, &N))) return rc;
    const int waves = whole_waves(s, prefix_lens, new_lens);   // the attention call's choice for launches it does not cut
    const int T = pbkv::attn_bf16_tile_tokens(s->head_dim, G, waves);
    *unit_tokens = T;
    std::vector<pbkv::TileDesc> &tiles = tl_tiles;
    if ((rc = build_tiles(s, prefix_lens, new_lens, blocks_bf16(s, waves), &tiles, pbkv::attn_bf16_units_per_tile(s->num_kv_heads, G),
                          waves == 4 ? 2 * MI355X_CUS : 0)))
        return rc;
    const int64_t units = (int64_t)tiles.size() * pbkv::attn_bf16_units_per_tile(s->num_kv_heads, G);
    *n_units = units;
    if (units == 0 || (!unit_xor && unit_capacity == 0)) return PBKV_OK;   // nothing to do / size query
    if (!unit_xor) return fail(PBKV_ERR_NULL, "pbkv_gather_probe: NULL unit_xor");
    if (unit_capacity < units)
        return fail(PBKV_ERR_RANGE, "pbkv_gather_probe: %lld units need room, unit_xor holds %lld", (long long)units,
                    (long long)unit_capacity);
    if ((rc = check_aligned(k_new, "k_new")) || (rc = check_aligned(v_new, "v_new")) ||
        (rc = check_aligned(kv_pool, "kv_pool")))
        return rc;
    if ((rc = check_device_ptr(k_new, "k_new")) || (rc = check_device_ptr(v_new, "v_new")) ||
        (rc = check_device_ptr(kv_pool, "kv_pool")) || (rc = check_device_ptr(block_table, "block_table")) ||
        (rc = check_device_ptr(unit_xor, "unit_xor")))
        return rc;

    if ((rc = check_not_capturing((hipStream_t)stream, "this call"))) return rc;
    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    Lease lease;
    if ((rc = ring_acquire(*ds, tiles.size() * sizeof(pbkv::TileDesc), &lease))) return rc;
    memcpy(lease.host, tiles.data(), tiles.size() * sizeof(pbkv::TileDesc));
    pbkv::AttnParams p;
    p.q = nullptr; p.k_new = k_new; p.v_new = v_new; p.kv_pool = kv_pool; p.out = unit_xor;
    p.block_table = block_table;
    p.tiles = (const pbkv::TileDesc *)lease.dev;
    p.n_tiles = (int32_t)tiles.size();
    p.Hq = s->num_q_heads; p.Hkv = s->num_kv_heads;
    p.max_pages = s->max_pages_per_req; p.num_pages = s->num_pages;
    p.waves = waves;
    p.mirror = nullptr; p.ranges = nullptr; p.mirror_ranges = nullptr; p.key_groups = 1; p.most_parts = 0; p.splits = 1; p.row_groups = 0;
    p.units = nullptr; p.mirror_units = nullptr; p.n_units = 0;
    p.merges = nullptr; p.mirror_merges = nullptr; p.n_merges = 0; p.partial = nullptr;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = pbkv::launch_gather_probe(p, s->head_dim, st);
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "gather probe launch");
    return rel;
}

int pbkv_append_kv(const pbkv_shape *s, const void *k_new, const void *v_new, void *kv_pool,
                   const int32_t *block_table, const int32_t *prefix_lens, const int32_t *new_lens,
                   void *stream) {
    g_err[0] = 0;
    int rc = check_shape(s, false);
    if (rc) return rc;
    if (s->batch == 0) return PBKV_OK;
    if (!k_new || !v_new || !kv_pool || !block_table || !prefix_lens || !new_lens)
        return fail(PBKV_ERR_NULL, "pbkv_append_kv: NULL argument");
    int64_t N = 0;
    if ((rc = check_lens(s, prefix_lens, new_lens, &N))) return rc;
    if (N == 0) return PBKV_OK;
    if ((rc = check_aligned(k_new, "k_new")) || (rc = check_aligned(v_new, "v_new")) ||
        (rc = check_aligned(kv_pool, "kv_pool")))
        return rc;
    if ((rc = check_device_ptr(k_new, "k_new")) || (rc = check_device_ptr(v_new, "v_new")) ||
        (rc = check_device_ptr(kv_pool, "kv_pool")) || (rc = check_device_ptr(block_table, "block_table")))
        return rc;

    hipStream_t st = (hipStream_t)stream;
    if ((rc = check_not_capturing(st, "pbkv_append_kv"))) return rc;
    pbkv::AppendParams p;
    p.k_new = k_new; p.v_new = v_new; p.kv_pool = kv_pool; p.block_table = block_table;
    p.mirror = nullptr;
    p.Hkv = s->num_kv_heads; p.max_pages = s->max_pages_per_req; p.num_pages = s->num_pages;

    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    StreamCache *sc = nullptr;
    char *slot = nullptr;
    if ((rc = stream_cache(*ds, st, true, &sc))) return rc;
    if (Plan *pl = find_plan(*ds, *sc, PLAN_APPEND, s, 0, prefix_lens, new_lens, &slot)) {
        p.descs = (const pbkv::AppendDesc *)slot;
        p.n_descs = pl->n_a;
        hipError_t e = pbkv::launch_append(p, s->head_dim, elt_bytes(s->dtype), st);
        return e == hipSuccess ? PBKV_OK : fail_hip(e, "append launch");
    }

    const int P = s->page_size;
    std::vector<pbkv::AppendDesc> &descs = tl_runs;
    descs.clear();
    int64_t row0 = 0;
    for (int r = 0; r < s->batch; r++) {
        const int64_t pr = prefix_lens[r], n = new_lens[r];
        for (int64_t t = 0; t < n;) {
            const int64_t pos = pr + t;
            const int slot0 = (int)(pos % P);
            const int count = (int)std::min<int64_t>(P - slot0, n - t);
            descs.push_back(pbkv::AppendDesc{row0 + t, r, (int32_t)(pos / P), slot0, count, 0});
            t += count;
        }
        row0 += n;
    }
    if (descs.size() > (size_t)INT32_MAX / 64) return fail(PBKV_ERR_LIMIT, "too many page runs");
    const size_t bytes = descs.size() * sizeof(pbkv::AppendDesc);
    Lease lease;
    if ((rc = ring_acquire(*ds, bytes, &lease))) return rc;
    memcpy(lease.host, descs.data(), bytes);
    p.descs = (const pbkv::AppendDesc *)lease.dev;
    p.n_descs = (int32_t)descs.size();
    Plan *pl = nullptr;
    if (bytes <= PLAN_SLOT_BYTES) {
        pl = new_plan(*ds, *sc, PLAN_APPEND, s, 0, prefix_lens, new_lens, &slot);
        pl->n_a = p.n_descs;
        p.mirror = (pbkv::AppendDesc *)slot;
    }
    hipError_t e = pbkv::launch_append(p, s->head_dim, elt_bytes(s->dtype), st);
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "append launch");
    if (pl) pl->valid = true;
    return rel;
}

}  // extern "C"

namespace {

// Page ids of a swap: inside the pool and (swap-in: they are destinations) all distinct.
int check_page_ids(const pbkv_shape *s, const int32_t *page_ids, int32_t n_pages, bool distinct) {
    for (int i = 0; i < n_pages; i++) {
        const int32_t id = page_ids[i];
        if (id < 0 || id >= s->num_pages)
            return fail(PBKV_ERR_RANGE, "page_ids[%d] = %d outside pool of %d pages", i, id, s->num_pages);
    }
    if (!distinct) return PBKV_OK;
    if ((int64_t)n_pages * 16 < s->num_pages) {
        // few pages of a large pool: sort a copy instead of clearing a flag per pool page
        std::vector<int32_t> &ids = tl_ids;
        ids.assign(page_ids, page_ids + n_pages);
        std::sort(ids.begin(), ids.end());
        for (int i = 1; i < n_pages; i++)
            if (ids[i] == ids[i - 1]) return fail(PBKV_ERR_ALIAS, "page id %d appears twice", ids[i]);
        return PBKV_OK;
    }
    std::vector<uint8_t> &seen = tl_seen;
    seen.assign((size_t)s->num_pages, 0);
    for (int i = 0; i < n_pages; i++) {
        const int32_t id = page_ids[i];
        if (seen[id]) return fail(PBKV_ERR_ALIAS, "page_ids[%d] = %d appears twice", i, id);
        seen[id] = 1;
    }
    return PBKV_OK;
}

}  // namespace

extern "C" {

int pbkv_swap_in_pages(const pbkv_shape *s, const void *host_pages, const int32_t *page_ids,
                       int32_t n_pages, void *kv_pool, void *stream) {
    g_err[0] = 0;
    int rc = check_shape(s, false);
    if (rc) return rc;
    if (n_pages < 0) return fail(PBKV_ERR_RANGE, "n_pages %d", n_pages);
    if (n_pages == 0) return PBKV_OK;
    if (!host_pages || !page_ids || !kv_pool) return fail(PBKV_ERR_NULL, "pbkv_swap_in_pages: NULL argument");
    if ((rc = check_page_ids(s, page_ids, n_pages, true))) return rc;
    if ((rc = check_aligned(host_pages, "host_pages")) || (rc = check_aligned(kv_pool, "kv_pool"))) return rc;
    const void *host_dev = nullptr;
    if ((rc = check_pinned_ptr(host_pages, "host_pages", &host_dev))) return rc;
    if ((rc = check_device_ptr(kv_pool, "kv_pool"))) return rc;

    if ((rc = check_not_capturing((hipStream_t)stream, "this call"))) return rc;
    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    Lease lease;
    if ((rc = ring_acquire(*ds, (size_t)n_pages * sizeof(int32_t), &lease))) return rc;
    memcpy(lease.host, page_ids, (size_t)n_pages * sizeof(int32_t));
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = pbkv::launch_swap_in(host_dev, (const int32_t *)lease.dev, n_pages, kv_pool,
                                        pbkv_page_bytes(s), st);
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "swap-in launch");
    return rel;
}

}  // extern "C"

namespace {

constexpr int64_t DECODE_TARGET_WGS = 2048;   // work-groups aimed for (1024 / 4096 / 8192 were measured: not faster)
constexpr int64_t DECODE_WHOLE_PAGES = 64;    // contexts that a large call leaves whole (figures: decode_cut)
constexpr int64_t DECODE_SHORT_PAGES = 5;     // contexts that every call leaves whole: the chain is shorter than any merge
// One kernel (the last work-group of a (request, KV head) merges) saves a launch, 3 us of host and GPU time, where the
// launch is short: 5000 tokens at 32/8 heads of 128 take 18.7 us against 20.4, 128 x (20 .. 300) at 32/2 22.5 against
// 27.5.  Its write-through stores cost a full chip more than that (300-us launches: +1 %), and one work-group
// is slow on many partials (32768 tokens at 32/2 heads: 73 us with all 128 slices merged by one, 26.5 by eight).
constexpr size_t DECODE_ONE_KERNEL_BYTES = 64u << 10;   // of partials that one work-group merges (what its threads hold, merge_held)
constexpr size_t STATIC_PARTIAL_BYTES = 8u << 20;   // of the entry point that allocates nothing
constexpr int STATIC_MAX_SLICES = 4096;
constexpr int STATIC_MAX_REQS = 4096;

// Validation shared by the decode entry points; also sums the pages of all contexts.
int check_decode_args(const pbkv_shape *s, const void *q, const void *kv_pool, const int32_t *block_table,
                      const int32_t *context_lens, void *out, int64_t *total_pages, const char *who) {
    int rc = check_shape(s, true);
    if (rc) return rc;
    if (s->dtype != PBKV_BF16) return fail(PBKV_ERR_DTYPE, "%s: bf16 only", who);
    *total_pages = 0;
    if (s->batch == 0) return PBKV_OK;
    if (!q || !kv_pool || !block_table || !context_lens || !out) return fail(PBKV_ERR_NULL, "%s: NULL argument", who);
    const int B = s->batch, P = s->page_size;
    for (int r = 0; r < B; r++) {
        const int64_t L = context_lens[r];
        if (L < 0 || L > INT32_MAX - 4096) return fail(PBKV_ERR_RANGE, "request %d: context length %lld", r, (long long)L);
        const int64_t pages = (L + P - 1) / P;
        if (pages > s->max_pages_per_req)
            return fail(PBKV_ERR_RANGE, "request %d needs %lld pages, block_table rows hold %d", r, (long long)pages,
                        s->max_pages_per_req);
        *total_pages += pages;
    }
    if ((rc = check_aligned(q, "q")) || (rc = check_aligned(kv_pool, "kv_pool")) || (rc = check_aligned(out, "out"))) return rc;
    if ((rc = check_device_ptr(q, "q")) || (rc = check_device_ptr(kv_pool, "kv_pool")) ||
        (rc = check_device_ptr(block_table, "block_table")) || (rc = check_device_ptr(out, "out")))
        return rc;
    return PBKV_OK;
}

// How a decode call's contexts are sliced.
struct DecodeCut {
    int32_t slice_pages;    // pages of a slice
    int32_t n_slices, n_parts;
    size_t scratch_bytes;
    bool one_kernel;        // the last work-group of a (request, KV head) merges the partials
    bool fits_static;       // pbkv_paged_decode_static takes the call
};

int64_t decode_parts(const pbkv_shape *s, const int32_t *context_lens, int64_t slice_pages, bool all) {
    int64_t n = 0;
    for (int r = 0; r < s->batch; r++) {
        const int64_t k = ((context_lens[r] + 15) / 16 + slice_pages - 1) / slice_pages;
        n += all || k > 1 ? k : 0;
    }
    return n;
}

// Large calls: enough work-groups to fill the chip a few times over, at least 16 pages each, or all contexts whole if none has more than
// DECODE_WHOLE_PAGES.  Up to there no call loses by it: us in slices and whole, 32/8 heads of 128: 66 x 1024 tokens 59, 56; 128 x 1024 91, 82; 512 x
// (16 .. 1024) 183, 186; 640 x (16 .. 1024) at 16/2 of 64 45, 42.  Past it calls of many contexts would gain still (128 x 1025 95, 84; 128 x 2000 168,
// 158; 400 x 1500 at 32/2 181, 117) and calls of fewer or uneven ones, which end on a chain of the longest one's pages, lose (66 x 1500 78, 81; 40 x 2000
// 60, 70; 100 x (16 .. 4096) 153, 172; 100 x (16 .. 2000) at 8/8 78, 90).  Smaller calls are weighed:
//   * a work-group's pages are a serial chain of fetches, 0.27 us each (0.32 and 0.4 with the arithmetic of 8 and 16 heads of 128);
//     work-groups that share a CU share its rate, at d = 64, half the bytes, two of them not yet;
//   * all pages pass through HBM, 0.34 us a page and CU at d = 128, half of that at 64;
//   * slices have to be merged, for 1.5 us and 7 ns per work-group that leaves a partial result, up to 512 of them, and 15 ns per
//     slice of the longest context; in a kernel of its own 3 us more.
// So short contexts stay whole where there are enough of them (us per call, in slices of 4 .. 16 pages -> whole, 32/8 heads of 128: 23 x 66
// tokens 10.6 -> 6.0, 16 x 250 11.6 -> 8.8, 64 x 500 37.0 -> 23.8, 52 x 827 42.7 -> 32.6), one of 250 tokens is cut in 4 (8.1 -> 7.4), and slices
// are longer where the chip is busy anyway (4 x 2000 tokens, of 8 -> 16 pages 14.5 -> 12.9; one of 16000, of 16 -> 32 20.9 -> 19.1).
// The limits of the entry point that allocates nothing are those of the large slices, and so is the slicing of a call
// whose partials would not fit there in small ones (its results are those of the other entry point, bit for bit).
int decode_cut(const pbkv_shape *s, const int32_t *context_lens, int64_t total_pages, DecodeCut *out) {
    const int G = s->num_q_heads / s->num_kv_heads, H = s->num_kv_heads;
    auto up4 = [](int64_t v) { return (v + 3) & ~(int64_t)3; };
    auto bytes = [&](int64_t parts) { return (size_t)(parts * H * pbkv::decode_partial_floats(s->head_dim, G)) * sizeof(float); };
    const int64_t wgs = total_pages * H;
    const int64_t large = std::max<int64_t>(16, up4((wgs * (G > 8 ? 2 : 1) + DECODE_TARGET_WGS - 1) / DECODE_TARGET_WGS));
    // (no more large slices than this; counted only where that may be past a limit)
    int64_t large_parts = total_pages / large + s->batch;
    if (large_parts > STATIC_MAX_SLICES || bytes(large_parts) > STATIC_PARTIAL_BYTES) large_parts = decode_parts(s, context_lens, large, true);
    if (large_parts > INT32_MAX / 64 - s->batch) return fail(PBKV_ERR_LIMIT, "too many slices");
    out->fits_static = large_parts <= STATIC_MAX_SLICES && bytes(std::max<int64_t>(large_parts, 1)) <= STATIC_PARTIAL_BYTES;
    int32_t longest = 1;
    for (int r = 0; r < s->batch; r++) longest = std::max(longest, (context_lens[r] + 15) / 16);
    int64_t pages = longest;
    if (wgs > 16 * DECODE_TARGET_WGS) {
        if (longest > DECODE_WHOLE_PAGES) pages = large;
    } else if (longest > DECODE_SHORT_PAGES) {
        const bool wide = s->head_dim == 128;
        const int64_t page = !wide || G <= 4 ? 270 : (G == 8 ? 320 : 400), through_hbm = wgs * (wide ? 344 : 172) / MI355X_CUS;       // ns
        auto time = [&](int64_t slice, int64_t n) {        // in n slices of up to so many pages (a CU with several gets some shorter ones)
            const int64_t on_cu = (n * H + MI355X_CUS - 1) / MI355X_CUS, shared = page * on_cu * (slice + total_pages / n) / 2;
            return std::max({page * slice, wide ? shared : shared / 2, through_hbm});
        };
        // slices of 4 .. 64 pages: how many, and how many of them leave a partial result
        constexpr int SIZES[] = {64, 48, 32, 24, 16, 12, 8, 4}, NS = sizeof SIZES / sizeof *SIZES;
        int32_t count[NS] = {}, parts[NS] = {};
        for (int r = 0; r < s->batch; r++) {
            const uint32_t n = ((uint32_t)context_lens[r] + 15) / 16;
#pragma unroll
            for (int k = 0; k < NS; k++) {
                const int32_t m = (int32_t)((n + SIZES[k] - 1) / SIZES[k]);
                count[k] += std::max(m, 1);
                parts[k] += m > 1 ? m : 0;
            }
        }
        int64_t best = time(longest, s->batch);
        for (int k = 0; k < NS; k++) {
            if (SIZES[k] >= longest) continue;
            const int64_t most = (longest + SIZES[k] - 1) / SIZES[k];
            const bool one_kernel = (int64_t)count[k] * H <= DECODE_ONE_KERNEL_WGS && bytes(most) / H <= DECODE_ONE_KERNEL_BYTES;
            const int64_t t = time(SIZES[k], count[k]) + 1500 + 7 * std::min<int64_t>((int64_t)parts[k] * H, 512) + 15 * most + (one_kernel ? 0 : 3000);
            if (t < best) {
                best = t;
                pages = SIZES[k];
            }
        }
    }
    int64_t parts = 0;
    if (pages < longest && bytes(parts = decode_parts(s, context_lens, pages, false)) > STATIC_PARTIAL_BYTES)
        parts = decode_parts(s, context_lens, pages = large, false);
    out->slice_pages = (int32_t)pages;
    out->n_parts = (int32_t)parts;
    out->n_slices = s->batch;
    int32_t most = 1;
    if (pages < longest) {
        out->n_slices = 0;
        for (int r = 0; r < s->batch; r++) {
            const int32_t k = std::max<int32_t>(1, ((context_lens[r] + 15) / 16 + out->slice_pages - 1) / out->slice_pages);
            out->n_slices += k;
            most = std::max(most, k);
        }
    }
    out->one_kernel = (int64_t)out->n_slices * H <= DECODE_ONE_KERNEL_WGS && bytes(most) / H <= DECODE_ONE_KERNEL_BYTES;
    out->scratch_bytes = bytes(parts);
    return PBKV_OK;
}

void fill_decode_reqs(const pbkv_shape *s, const int32_t *context_lens, int32_t slice_pages, pbkv::DecodeReq *reqs) {
    int32_t slice = 0, part = 0;
    for (int r = 0; r < s->batch; r++) {
        const int32_t k = std::max<int32_t>(1, ((context_lens[r] + 15) / 16 + slice_pages - 1) / slice_pages);
        reqs[r] = pbkv::DecodeReq{context_lens[r], slice, part};
        slice += k;
        part += k > 1 ? k : 0;
    }
}

pbkv::DecodeParams decode_params(const pbkv_shape *s, const void *q, const void *kv_pool, const int32_t *block_table, void *out) {
    pbkv::DecodeParams p{};
    p.q = q; p.kv_pool = kv_pool; p.out = out; p.block_table = block_table;
    p.n_reqs = s->batch;
    p.Hq = s->num_q_heads; p.Hkv = s->num_kv_heads;
    p.max_pages = s->max_pages_per_req; p.num_pages = s->num_pages;
    return p;
}

}  // namespace

extern "C" {

int pbkv_paged_decode(const pbkv_shape *s, const void *q, const void *kv_pool, const int32_t *block_table,
                      const int32_t *context_lens, void *out, void *stream) {
    g_err[0] = 0;
    int64_t total_pages = 0;
    int rc = check_decode_args(s, q, kv_pool, block_table, context_lens, out, &total_pages, "pbkv_paged_decode");
    if (rc) return rc;
    if (s->batch == 0) return PBKV_OK;
    hipStream_t st = (hipStream_t)stream;
    if ((rc = check_not_capturing(st, "pbkv_paged_decode"))) return rc;
    pbkv::DecodeParams p = decode_params(s, q, kv_pool, block_table, out);
    pbkv::DecodeList inl;

    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    StreamCache *sc = nullptr;
    char *slot = nullptr;
    if ((rc = stream_cache(*ds, st, true, &sc))) return rc;
    const bool listed = s->batch > pbkv::DECODE_INLINE_REQS;
    if (Plan *pl = listed ? find_plan(*ds, *sc, PLAN_DECODE, s, 0, context_lens, nullptr, &slot) : nullptr) {
        if ((rc = stream_scratch(*sc, (size_t)pl->aux, true, &p.scratch))) return rc;
        p.reqs = (const pbkv::DecodeReq *)slot;
        p.n_slices = pl->n_a;
        p.slice_pages = pl->n_b;
        if (pl->waves) decode_counters(*sc, &p.counters);
        hipError_t e = pbkv::launch_decode_bf16(p, inl, s->head_dim, st);
        return e == hipSuccess ? PBKV_OK : fail_hip(e, "decode launch");
    }

    DecodeCut cut;
    if ((rc = decode_cut(s, context_lens, total_pages, &cut))) return rc;
    if ((rc = stream_scratch(*sc, cut.scratch_bytes, true, &p.scratch))) return rc;
    if (cut.one_kernel) decode_counters(*sc, &p.counters);
    p.n_slices = cut.n_slices;
    p.slice_pages = cut.slice_pages;
    if (!listed) {
        fill_decode_reqs(s, context_lens, cut.slice_pages, inl.r);
        hipError_t e = pbkv::launch_decode_bf16(p, inl, s->head_dim, st);
        return e == hipSuccess ? PBKV_OK : fail_hip(e, "decode launch");
    }

    std::vector<pbkv::DecodeReq> &reqs = tl_reqs;
    reqs.resize((size_t)s->batch);
    fill_decode_reqs(s, context_lens, cut.slice_pages, reqs.data());
    const size_t bytes = reqs.size() * sizeof(pbkv::DecodeReq);
    Lease lease;
    if ((rc = ring_acquire(*ds, bytes, &lease))) return rc;
    memcpy(lease.host, reqs.data(), bytes);
    p.reqs = (const pbkv::DecodeReq *)lease.dev;
    Plan *pl = nullptr;
    if (bytes <= PLAN_SLOT_BYTES) {
        pl = new_plan(*ds, *sc, PLAN_DECODE, s, 0, context_lens, nullptr, &slot);
        pl->n_a = p.n_slices;
        pl->n_b = p.slice_pages;
        pl->waves = cut.one_kernel;
        pl->aux = (int64_t)cut.scratch_bytes;
        p.mirror_reqs = (pbkv::DecodeReq *)slot;
    }
    hipError_t e = pbkv::launch_decode_bf16(p, inl, s->head_dim, st);
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "decode launch");
    if (pl) pl->valid = true;
    return rel;
}

int pbkv_swap_out_pages(const pbkv_shape *s, const void *kv_pool, const int32_t *page_ids,
                        int32_t n_pages, void *host_pages, void *stream) {
    g_err[0] = 0;
    int rc = check_shape(s, false);
    if (rc) return rc;
    if (n_pages < 0) return fail(PBKV_ERR_RANGE, "n_pages %d", n_pages);
    if (n_pages == 0) return PBKV_OK;
    if (!host_pages || !page_ids || !kv_pool) return fail(PBKV_ERR_NULL, "pbkv_swap_out_pages: NULL argument");
    if ((rc = check_page_ids(s, page_ids, n_pages, false))) return rc;
    if ((rc = check_aligned(host_pages, "host_pages")) || (rc = check_aligned(kv_pool, "kv_pool"))) return rc;
    const void *host_dev = nullptr;
    if ((rc = check_pinned_ptr(host_pages, "host_pages", &host_dev))) return rc;
    if ((rc = check_device_ptr(kv_pool, "kv_pool"))) return rc;

    if ((rc = check_not_capturing((hipStream_t)stream, "this call"))) return rc;
    DevState *ds = nullptr;
    if ((rc = device_state(&ds))) return rc;
    std::lock_guard<std::mutex> lock(ds->mu);
    Lease lease;
    if ((rc = ring_acquire(*ds, (size_t)n_pages * sizeof(int32_t), &lease))) return rc;
    memcpy(lease.host, page_ids, (size_t)n_pages * sizeof(int32_t));
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = pbkv::launch_swap_out(kv_pool, (const int32_t *)lease.dev, n_pages, (void *)host_dev,
                                         pbkv_page_bytes(s), st);
    int rel = ring_release(lease, st);
    if (e != hipSuccess) return fail_hip(e, "swap-out launch");
    return rel;
}

}  // extern "C"

// ---- decode without any allocation -----------------------------------------------------------
// For callers that cannot allocate device memory (code under graph capture, tight serving loops,
// harnesses that forbid it): the partials of the context slices and the list of a call of many requests live in
// one file-scope device array instead of library-allocated buffers, and the list reaches the kernels through
// kernel arguments (a launch copies its arguments before it returns, so no host buffer has to stay
// alive and no ring, event or copy is involved).  The partials are merged by a second kernel: counters for the
// one-kernel form would be left wrong for good by two calls that overlap, which here only spoil each other's results.
namespace {

constexpr size_t STATIC_REQS_OFF = STATIC_PARTIAL_BYTES;
constexpr size_t STATIC_BYTES = STATIC_REQS_OFF + STATIC_MAX_REQS * sizeof(pbkv::DecodeReq);

// Every GPU the library runs on holds its own copy of this array, at its own address, until the
// process ends.  In host code the name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[STATIC_BYTES];

std::mutex g_static_mu;
void *g_static_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device (asked once per device).
int static_scratch(unsigned char **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(PBKV_ERR_DEVICE, "device index %d unsupported", dev);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return fail_hip(e, "hipGetSymbolAddress(scratch)");
        g_static_ptr[dev] = ptr;
    }
    *out = (unsigned char *)g_static_ptr[dev];
    return PBKV_OK;
}

constexpr int STAGE_WORDS = 896;                     // 3.5 KiB of a launch's 4 KiB of arguments
struct StageChunk { uint32_t w[STAGE_WORDS]; };

__global__ __launch_bounds__(256) void stage_kernel(StageChunk c, uint32_t *dst, int n) {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = c.w[i];
}

// Copies `bytes` (a multiple of 4) of host memory to device memory at dst through kernel arguments.
hipError_t stage_words(const void *src, size_t bytes, void *dst, hipStream_t st) {
    const uint32_t *w = (const uint32_t *)src;
    size_t words = bytes / 4;
    uint32_t *d = (uint32_t *)dst;
    while (words > 0) {
        const int n = (int)std::min<size_t>(words, STAGE_WORDS);
        StageChunk c;
        memcpy(c.w, w, (size_t)n * 4);
        hipLaunchKernelGGL(stage_kernel, dim3(1), dim3(256), 0, st, c, d, n);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        w += n;
        d += n;
        words -= n;
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

int pbkv_paged_decode_static(const pbkv_shape *s, const void *q, const void *kv_pool, const int32_t *block_table,
                             const int32_t *context_lens, void *out, void *stream) {
    g_err[0] = 0;
    int64_t total_pages = 0;
    int rc = check_decode_args(s, q, kv_pool, block_table, context_lens, out, &total_pages, "pbkv_paged_decode_static");
    if (rc) return rc;
    if (s->batch == 0) return PBKV_OK;
    if (s->batch > STATIC_MAX_REQS)
        return fail(PBKV_ERR_LIMIT, "pbkv_paged_decode_static: %d requests, at most %d", s->batch, STATIC_MAX_REQS);
    DecodeCut cut;
    if ((rc = decode_cut(s, context_lens, total_pages, &cut))) return rc;
    if (!cut.fits_static)
        return fail(PBKV_ERR_LIMIT, "pbkv_paged_decode_static: more than %d context slices or %zu bytes of partial results",
                    STATIC_MAX_SLICES, STATIC_PARTIAL_BYTES);
    unsigned char *base = nullptr;
    if ((rc = static_scratch(&base))) return rc;

    hipStream_t st = (hipStream_t)stream;
    pbkv::DecodeParams p = decode_params(s, q, kv_pool, block_table, out);
    pbkv::DecodeList inl;
    p.scratch = (float *)base;
    p.n_slices = cut.n_slices;
    p.slice_pages = cut.slice_pages;
    hipError_t e;
    if (s->batch <= pbkv::DECODE_INLINE_REQS) {
        fill_decode_reqs(s, context_lens, cut.slice_pages, inl.r);
    } else {
        std::vector<pbkv::DecodeReq> &reqs = tl_reqs;
        reqs.resize((size_t)s->batch);
        fill_decode_reqs(s, context_lens, cut.slice_pages, reqs.data());
        e = stage_words(reqs.data(), reqs.size() * sizeof(pbkv::DecodeReq), base + STATIC_REQS_OFF, st);
        if (e != hipSuccess) return fail_hip(e, "work-list launch");
        p.reqs = (const pbkv::DecodeReq *)(base + STATIC_REQS_OFF);
    }
    e = pbkv::launch_decode_bf16(p, inl, s->head_dim, st);
    return e == hipSuccess ? PBKV_OK : fail_hip(e, "decode launch");
}

}  // extern "C"

