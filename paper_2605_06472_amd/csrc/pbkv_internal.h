// Internal declarations shared by the host API and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbkv {

// Sets the thread's last-error text (returned by pbkv_last_error) and hands back `code`.
int set_error(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// One unit of attention work: a block of consecutive suffix tokens of one request.
// Written by the host into pinned memory and read by the kernel through the mapped
// pointer (32 bytes, two 16-byte loads).
struct TileDesc {
    int32_t req;         // request index inside this call (row of block_table)
    int32_t tok0;        // first suffix token of the tile (fp32: first row, a row being a token's query head of the group)
    int32_t prefix_len;  // p_r
    int32_t new_len;     // n_r
    int64_t row0;        // packed row (into q / k_new / v_new / out) of the request's token 0
    int64_t index;       // index of the token block in request order (before the longest-first sort)
};
static_assert(sizeof(TileDesc) == 32, "TileDesc is read as two 16-byte words");

// The KV tiles a unit takes of those its tokens attend to, in launches that deal them out to several units (16
// bytes beside the tile, so that the list of a launch without ranges is no longer than before there were any).
struct RangeDesc {
    int32_t part;        // number of the partial result, or -1: the range is the whole context and the unit
                         // writes `out` itself
    int32_t kt0, kt1;    // KV tiles [kt0, kt1) of the token block; tiles past the block's last one count as none.
                         // bf16: 64 keys each, the prefix's (the last may be partial), then the suffix's; fp32: 32
                         // keys each, numbered through prefix and suffix
    int32_t slot;        // where the partial result stands in AttnParams::partial: a slot is a work-group of all KV heads, and
                         // a part has as many as its token block has work-groups with rows (fp32: one, so slot = part)
};
static_assert(sizeof(RangeDesc) == 16, "RangeDesc is read as one 16-byte word");

// A token block whose KV tiles were dealt out to several units: where their partial results stand.
struct MergeDesc {
    int32_t tok0, new_len;
    int32_t part0, n_parts;   // partial results part0 .. part0 + n_parts - 1
    int64_t row0;
    int32_t slot0, splits;    // slot of the first, slots of each
};
static_assert(sizeof(MergeDesc) == 32, "MergeDesc is read as two 16-byte words");

// A run of consecutive suffix tokens of one request that land in one pool page.
struct AppendDesc {
    int64_t src_row;     // packed row of the first token of the run
    int32_t req;         // request index (row of block_table)
    int32_t logical_page;
    int32_t slot0;       // first slot inside the page
    int32_t count;       // tokens in the run (1..page_size)
    int64_t pad;
};
static_assert(sizeof(AppendDesc) == 32, "AppendDesc is read as two 16-byte words");

struct AttnParams {
    const void *q, *k_new, *v_new, *kv_pool;
    void *out;
    const int32_t *block_table;
    const TileDesc *tiles;
    int32_t n_tiles, Hq, Hkv, max_pages, num_pages;
    int32_t waves;   // bf16 kernel: waves per work-group (attn_bf16_waves); the tiles were cut for it
    int32_t key_groups;   // bf16 kernel, 4 waves: 1, or 2 for work-groups of twice four waves that share a unit's KV tiles out
    TileDesc *mirror;   // device memory that receives a copy of the tiles the launch read, or null
    const RangeDesc *ranges;   // [n_tiles], or null: every unit takes all tiles of its tokens
    RangeDesc *mirror_ranges;
    const MergeDesc *merges;   // token blocks with partial results (n_merges of them; 0: no second kernel)
    MergeDesc *mirror_merges;
    int32_t n_merges;
    int32_t most_parts;   // of one token block
    int32_t splits;     // bf16: work-groups of a tile per KV head (attn_bf16_splits), of the longest request's
    int32_t row_groups; // bf16: 32-row groups of a token block that the second kernel looks at: no block has rows in more
    float *partial;     // the partial results
    // (behind the rest, so that what every work-group begins with stays in one line of arguments: two cost short launches 0.16 us)
    const uint32_t *units;    // bf16: 4 * tile + work-group of the tile, of all that hold rows, or null: `splits` of every tile
    uint32_t *mirror_units;
    int32_t n_units;    // ... of them per KV head
};

// Decode: a request, its first slice (slices are numbered over the whole call; a request without context has
// one too) and the slot of its first partial result (requests of one slice have none).
struct DecodeReq { int32_t ctx_len, slice0, part0; };
static_assert(sizeof(DecodeReq) == 12, "three words");

// Calls of up to this many requests pass their list as a kernel argument (1.5 KiB of at most 4): nothing is
// built, copied or cached for them.  A list in device memory is read 1 % faster in a long launch, and costs a first
// pass 7 us more.
constexpr int DECODE_INLINE_REQS = 128;
struct DecodeList { DecodeReq r[DECODE_INLINE_REQS]; };

struct DecodeParams {
    const void *q, *kv_pool;
    void *out;
    const int32_t *block_table;
    const DecodeReq *reqs;      // null: the list is the kernel argument
    DecodeReq *mirror_reqs;     // device memory that receives a copy of reqs, or null
    float *scratch;
    uint32_t *counters;         // [n_reqs][Hkv], zero between launches; null: a second kernel merges the partials
    int32_t n_slices, n_reqs, slice_pages, Hq, Hkv, max_pages, num_pages;
};

struct AppendParams {
    const void *k_new, *v_new;
    void *kv_pool;
    const int32_t *block_table;
    const AppendDesc *descs;
    AppendDesc *mirror;         // device memory that receives a copy of descs, or null
    int32_t n_descs, Hkv, max_pages, num_pages;
};

// Waves per work-group the bf16 kernel runs this batch with, and the tokens per attention tile
// that follow from it (what the host cuts the suffix into).
int attn_bf16_waves(const int32_t *prefix_lens, const int32_t *new_lens, int batch);
void attn_bf16_force_waves(int waves);   // 4 or 8: every later launch uses that shape; anything else: automatic
int attn_bf16_forced_waves();
int attn_bf16_tile_tokens(int head_dim, int group, int waves);
constexpr int KV_TILE = 64;    // keys per tile step of the bf16 attention kernels
constexpr int F32_KEYS = 32;   // ... and of the fp32 one
int attn_f32_block_rows();    // fp32: (token, query head of the group) rows per work-group
int64_t attn_f32_partial_floats(int head_dim);
int64_t attn_bf16_partial_floats(int head_dim);   // floats one work-group's partial result occupies (4-wave shape)

// Launchers: all arguments already validated.  Return the hipError of the launch.
hipError_t launch_attn_bf16(const AttnParams &p, int head_dim, hipStream_t s);
hipError_t launch_attn_f32(const AttnParams &p, int head_dim, hipStream_t s);
// Gather diagnostic: p.out is a uint32 array with one word per work unit, units ordered
// (tile in request order, query-head split, KV head); attn_bf16_units_per_tile gives the
// number of units of one tile.
hipError_t launch_gather_probe(const AttnParams &p, int head_dim, hipStream_t s);
int attn_bf16_units_per_tile(int num_kv_heads, int group);
int attn_bf16_splits(int group, int waves, int tokens);
hipError_t launch_append(const AppendParams &p, int head_dim, int elt_bytes, hipStream_t s);
hipError_t launch_swap_in(const void *host_pages, const int32_t *page_ids_dev, int32_t n_pages,
                          void *kv_pool, int64_t page_bytes, hipStream_t s);

// Paged decode attention (bf16).
hipError_t launch_decode_bf16(const DecodeParams &p, const DecodeList &inl, int head_dim, hipStream_t s);
int64_t decode_partial_floats(int head_dim, int group);   // floats one work-group's partial occupies
hipError_t launch_clear_words(uint32_t *w, int n, hipStream_t s);

hipError_t launch_swap_out(const void *kv_pool, const int32_t *page_ids_dev, int32_t n_pages,
                           void *host_pages, int64_t page_bytes, hipStream_t s);

// Fold of n partial results by one lane: part i has (reference, row sum) at ml + i * stride and a run of
// unnormalised output (Vec) at po + i * stride.  num = sum of exp2(reference_i - M) o_i, den the same of the row sums,
// added in the order of i.  The kernels around it are short and bound by dependent fetches from another XCD's
// stores: everything of the first AHEAD parts is loaded before the first use, so that up to that many parts take one
// round trip.  With a loop for M and one for the sums, eight parts at a time, they took four: 12001 + 37 tokens, 32/8
// heads of 128, 16 parts, with append 28.8 -> 25.5 us per pass.
constexpr int MERGE_AHEAD = 16;     // what cut launches aim at, where their ranges are short
#if defined(__HIP__)      // the host-only policy core includes this header too
template <int AHEAD, class Vec>
__device__ __forceinline__ void merge_parts(const float *ml, const float *po, int64_t stride, int n, Vec &num, float &den) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    constexpr int W = sizeof(Vec) / 4;
    f32x2 x[AHEAD];
    Vec o[AHEAD];
    auto load = [&](int i0) {
#pragma unroll
        for (int k = 0; k < AHEAD; k++) {
            x[k] = f32x2{-INFINITY, 0.f};                         // past the end: counts nothing
#pragma unroll
            for (int e = 0; e < W; e++) o[k][e] = 0.f;
            if (i0 + k < n) {                                     // uniform
                x[k] = *(const f32x2 *)(ml + (i0 + k) * stride);
                o[k] = *(const Vec *)(po + (i0 + k) * stride);
            }
        }
    };
    load(0);
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < AHEAD; k++) M = fmaxf(M, x[k][0]);
#pragma unroll 8
    for (int i = AHEAD; i < n; i++) M = fmaxf(M, ml[i * stride]);
#pragma unroll
    for (int e = 0; e < W; e++) num[e] = 0.f;
    den = 0.f;
    for (int i0 = 0; i0 < n; i0 += AHEAD) {
        if (i0 > 0) load(i0);
#pragma unroll
        for (int k = 0; k < AHEAD; k++) {
            const float f = __builtin_amdgcn_exp2f(x[k][0] - M);
            den = fmaf(f, x[k][1], den);
#pragma unroll
            for (int e = 0; e < W; e++) num[e] = fmaf(f, o[k][e], num[e]);
        }
    }
}
#endif

}  // namespace pbkv
