// Paged decode attention, bf16 (one query row per request over its paged context): the
// pure-decode step behind which prefetch transfers are hidden.  HBM-bound: every K and V row of
// the context is read exactly once, 4 KiB at a time, and nothing else of size moves.
//
// Work decomposition
//   work-group = 4 waves = (request, slice of its pages, KV head), all query heads of the group.
//   A wave takes every fourth page of the slice and keeps the K and V rows of the NEXT page in
//   flight (in registers) while it works on the current one: 8 KiB per wave, 64 per CU, enough
//   outstanding bytes to cover the HBM latency.  No LDS traffic and no barrier inside the loop.
//   The slice's request is found from the list of first slices, which comes as a kernel argument
//   (up to DECODE_INLINE_REQS requests): no work list is built, staged or read through a pointer.  It is read with the other
//   arguments, by kernels of their own: behind a branch on where the list is, the compiler puts its loads after the wait
//   for the arguments, and in a search the context length after that (us, that way -> now: 16 x 40 tokens at 32/8 heads of 128 4.3 -> 4.0,
//   65 x 64 at 16/2 of 64 4.2 -> 3.8, one of 1003 at 32/8 7.9 -> 7.6).
//   How long a slice is: decode_cut on the host side, with figures; a context that stays whole needs no merge.
//
//   scores     S[token][head] = K Q^T on the 16x16x32 bf16 MFMA: the A operand (16 tokens x 32 d)
//              is exactly 16 bytes per lane of a row-major K page, so K goes from global memory
//              into the MFMA without any shuffle; the query heads of the GQA group are the columns.
//   softmax    the 16-lane group g owns tokens 4g..4g+3 of the page (that is where the MFMA leaves
//              their scores); one reference maximum per head for the whole wave, moved only when a
//              score exceeds it by 2^8.
//   P V        in fp32, so the probabilities stay fp32: lane (g, c) loads d-values E*c.. of its group's tokens, widened from
//              bf16, and holds the probabilities of these tokens for head c, which are an fp32 MFMA's operands as they stand.
//              Up to 8 heads the 4x4x1 of 16 blocks: a block is four d of one lane group's token, the probabilities
//              of four heads are broadcast to the group's blocks, each group sums its own tokens and the four
//              meet once, at the end.  It takes 8 clocks for what the 16x16x4, 12 of whose 16 columns are empty at 4
//              heads, takes 32: 16 requests of 4000 tokens, 32/8 heads of 128, 55.4 -> 51.4 us, 41 of 4494 128.5 -> 122, 64 of
//              1024 .. 16384 (HBM-bound, 6.2 TB/s) 362.9 -> 357.8; at 8 heads of 64 16 x 4000 13.6 -> 12.9, 100 x 300 7.4 -> 7.2.  16 heads fill the 16x16x4, O^T[d][head] = V^T P^T (A row c is
//              d = E*c + e of the e-th product).
//   occupancy  two work-groups per CU at d = 128 (three: 9 % slower on the large batches, as are three page
//              buffers by 2 %), four at d = 64, whose pages are half the size (two: 98 us, four: 91 on 100 x 4/4
//              heads of 3000 .. 6000 tokens).
//   The four waves merge their partials (reference, row sum, unnormalised output) in LDS.  A request of
//   one slice is finished there; of a longer one the work-group writes a partial to a scratch buffer, and
//   the last work-group of a (request, KV head) merges them (fused form), or a second small kernel does.
#include "pbkv_internal.h"

#include <algorithm>

namespace pbkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr int DEC_WAVES = 4;
constexpr int DEC_THREADS = 64 * DEC_WAVES;
[[maybe_unused]] constexpr int DEC_MAX_HEADS = 16;                       // query heads per KV head: the MFMA's columns
[[maybe_unused]] constexpr float DEC_RESCALE_LOG2 = 8.0f;

constexpr int MERGE_ITEMS = 64;                         // groups of four output values a merging work-group takes at once
[[maybe_unused]] constexpr int MERGE_WEIGHTS = 2048;                     // (slice, head) weights it holds in LDS
static int merge_chunks(int head_dim, int group) { return std::max(1, group * head_dim / 4 / MERGE_ITEMS); }

template <int I> struct IntC { static constexpr int value = I; };

// floats per partial: [G][D] output, [G] (reference, row sum), padded to 16 bytes
int64_t decode_partial_floats(int head_dim, int group) { return ((int64_t)group * (head_dim + 2) + 3) & ~(int64_t)3; }

// The V values a lane takes of one token: E consecutive ones in E/2 words.
template <int D> struct VRow;
template <> struct VRow<128> { typedef u32x4 type; };
template <> struct VRow<64> { typedef u32x2 type; };

#if defined(__HIP_DEVICE_COMPILE__)
// exp2(m - ref) where m == -inf counts nothing (a wave without pages)
static __device__ __forceinline__ float weight(float m, float ref) { return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - ref); }

// x of this lane and of the lane 32 (16) away, added; lanes whose bit 5 (bit 4) is set get the sum of y instead.
static __device__ __forceinline__ float fold32(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
static __device__ __forceinline__ float fold16(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Over the lanes of a head, which differ in the bits from G up (G a power of two to 16), in every one of them: by exchanges
// inside the vector ALU, where a shuffle goes through LDS (their chain was a sixth of a merge's clocks behind its loads).
template <class Fold>
static __device__ __forceinline__ float over_head(float v, int G, Fold &&fold) {
    auto ror = [&](auto ctrl) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false)); };
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fold(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fold(__uint_as_float(b[0]), __uint_as_float(b[1]));
    if (G <= 8) v = fold(v, ror(IntC<0x128>{}));           // rotations inside a row of 16 lanes by 8, 4, 2, 1
    if (G <= 4) v = fold(v, ror(IntC<0x124>{}));
    if (G <= 2) v = fold(v, ror(IntC<0x122>{}));
    if (G <= 1) v = fold(v, ror(IntC<0x121>{}));
    return v;
}
static __device__ __forceinline__ float max_over_head(float v, int G) {
    return over_head(v, G, [](float x, float y) { return fmaxf(x, y); });
}
static __device__ __forceinline__ float sum_over_head(float v, int G) {
    return over_head(v, G, [](float x, float y) { return x + y; });
}

// Two neighbouring floats of a partial.  WRITE_THROUGH: past this XCD's L2, for a reader on another one.
template <bool WRITE_THROUGH>
static __device__ __forceinline__ void store_partial(float *dst, float a, float b) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    const f32x2 v = {a, b};
    if constexpr (WRITE_THROUGH) {
        uint64_t u;
        __builtin_memcpy(&u, &v, 8);
        __hip_atomic_store((uint64_t *)dst, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        *(f32x2 *)dst = v;
    }
}

// Merge of the partials of one (request, KV head), normalised and rounded once to bf16, by the threads of a work-group of
// DEC_THREADS.  `base` is slice 0's partial, `stride` the floats between slices.  Which of the two forms below
// serves a (n, G, D) follows from these alone, and so does the order of every sum: the kernel that merges
// does not show in the result.
//
// Up to MERGE_HELD groups of four output values in all (64 KiB of partials, every merge of the one-kernel form): the
// threads load everything at once, 16 groups and one (reference, row sum) each, and weigh what they
// hold: one trip to the other XCDs' stores, which is what a merge of this size costs.  (With references, weights and
// outputs fetched one after the other, 64 output groups at a time, the merge of 16 slices of 4 heads of 128
// took 12000 of a work-group's 22000 clocks: one request of 1003 tokens with append 13.8 -> 11.3 us per pass, 24 of up to
// 4097 at 16/2 heads of 64, where a second kernel merges, 17.7 -> 16.7.)
constexpr int MERGE_HELD = 16 * DEC_THREADS;
template <int D>
static __device__ __forceinline__ void merge_held(const float *base, int64_t stride, int n, int G, __bf16 *out) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    __shared__ float red_m[DEC_WAVES][DEC_MAX_HEADS], red_d[DEC_WAVES][DEC_MAX_HEADS];
    __shared__ float wt[DEC_THREADS];                  // [slice][head]; n * G is at most MERGE_HELD * 4 / D <= 256
    __shared__ __attribute__((aligned(16))) f32x4 red_o[DEC_THREADS];
    const int tid = threadIdx.x;
    const int items = G * D / 4, shift = __builtin_ctz(items), total = n * items;   // a power of two, 16 .. 512
    f32x4 x[MERGE_HELD / DEC_THREADS];
#pragma unroll
    for (int k = 0; k < MERGE_HELD / DEC_THREADS; k++) {
        const int e = k * DEC_THREADS + tid;           // (slice, group)
        x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (e < total) x[k] = *(const f32x4 *)(base + (e >> shift) * stride + (e & (items - 1)) * 4);
    }
    const int h = tid & (G - 1);                       // G divides 64: lanes of one head differ in the bits above G
    f32x2 ml = {-INFINITY, 0.f};
    if (tid / G < n) ml = *(const f32x2 *)(base + (tid / G) * stride + G * D + 2 * h);
    const float m = max_over_head(ml[0], G);
    if ((tid & 63) < G) red_m[tid >> 6][h] = m;
    __syncthreads();
    static_assert(DEC_WAVES == 4, "folds four");
    const float f = weight(ml[0], fmaxf(fmaxf(red_m[0][h], red_m[1][h]), fmaxf(red_m[2][h], red_m[3][h])));
    wt[tid] = f;
    const float d = sum_over_head(f * ml[1], G);
    if ((tid & 63) < G) red_d[tid >> 6][h] = d;
    __syncthreads();
    auto store = [&](int it, const f32x4 &o) {
        const int ho = it * 4 / D;
        const float den = (red_d[0][ho] + red_d[1][ho]) + (red_d[2][ho] + red_d[3][ho]);
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; e++) r[e] = (__bf16)(den > 0.f ? o[e] / den : 0.f);
        *(bf16x4 *)(out + it * 4) = r;
    };
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};      // 512 groups: two per thread; fewer: two chains
#pragma unroll
    for (int k = 0; k < MERGE_HELD / DEC_THREADS; k++) {
        if (k * DEC_THREADS >= total) break;           // uniform
        const int e = k * DEC_THREADS + tid;
        const float we = wt[(e >> shift) * G + (e & (items - 1)) * 4 / D];
#pragma unroll
        for (int c = 0; c < 4; c++) acc[k & 1][c] = fmaf(we, x[k][c], acc[k & 1][c]);
    }
    if (items > DEC_THREADS) {
        store(tid, acc[0]);
        store(tid + DEC_THREADS, acc[1]);
        return;
    }
    f32x4 o = acc[0] + acc[1];
    if (items < DEC_THREADS) {
        red_o[tid] = o;
        __syncthreads();
        if (tid >= items) return;
        for (int k = items + tid; k < DEC_THREADS; k += items) o += red_o[k];
    }
    store(tid, o);
}

// Larger ones, by several work-groups: chunk `chunk` of the output, MERGE_ITEMS groups of four values (or all, if
// there are fewer).
template <int D>
static __device__ __forceinline__ void merge_slices(const float *base, int64_t stride, int n, int G, int chunk, __bf16 *out) {
    __shared__ float red_m[DEC_WAVES][DEC_MAX_HEADS], red_d[DEC_WAVES][DEC_MAX_HEADS];
    __shared__ float wt[MERGE_WEIGHTS];
    __shared__ __attribute__((aligned(16))) f32x4 red_o[DEC_THREADS];
    const int tid = threadIdx.x;
    {
        const int h = tid % G;                         // G divides 64: lanes of one head differ in the bits above G
        float m = -INFINITY, d = 0.f;
#pragma unroll 4
        for (int s = tid / G; s < n; s += DEC_THREADS / G) {
            const float *ps = base + s * stride + G * D + 2 * h;
            const float ms = ps[0], ds = ps[1], nm = fmaxf(m, ms);
            d = d * weight(m, nm) + ds * weight(ms, nm);
            m = nm;
        }
        for (int x = 32; x >= G; x >>= 1) {
            const float mo = __shfl_xor(m, x, 64), od = __shfl_xor(d, x, 64), nm = fmaxf(m, mo);
            d = d * weight(m, nm) + od * weight(mo, nm);
            m = nm;
        }
        if ((tid & 63) < G) {
            red_m[tid >> 6][h] = m;
            red_d[tid >> 6][h] = d;
        }
    }
    __syncthreads();
    auto reference = [&](int h) { return fmaxf(fmaxf(red_m[0][h], red_m[1][h]), fmaxf(red_m[2][h], red_m[3][h])); };
    static_assert(DEC_WAVES == 4, "reference() folds four");
    const int items = min(G * D / 4, MERGE_ITEMS), ng = DEC_THREADS / items;     // ng threads share an item's slices
    const int per_block = MERGE_WEIGHTS / G;                                     // slices whose weights fit in LDS
    const int grp = tid / items;
    const int it = chunk * items + tid % items, h = it * 4 / D;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < n; s0 += per_block) {
        const int s1 = min(n, s0 + per_block);
        if (s0 > 0) __syncthreads();
        for (int i = tid; i < (s1 - s0) * G; i += DEC_THREADS)
            wt[i] = weight(base[(s0 + i / G) * stride + G * D + 2 * (i % G)], reference(i % G));
        __syncthreads();
#pragma unroll 8
        for (int s = s0 + grp; s < s1; s += ng) {
            const f32x4 x = *(const f32x4 *)(base + s * stride + it * 4);
            const float f = wt[(s - s0) * G + h];
#pragma unroll
            for (int e = 0; e < 4; e++) o[e] = fmaf(f, x[e], o[e]);
        }
    }
    red_o[tid] = o;
    __syncthreads();
    if (grp == 0) {
        for (int k = 1; k < ng; k++)
#pragma unroll
            for (int e = 0; e < 4; e++) o[e] += red_o[k * items + tid][e];
        const float M = reference(h);
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; w++) den += red_d[w][h] * weight(red_m[w][h], M);
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; e++) r[e] = (__bf16)(den > 0.f ? o[e] / den : 0.f);
        *(bf16x4 *)(out + it * 4) = r;
    }
}

// Request that slice `u` belongs to: the last one whose first slice is not behind it.  The whole wave looks at 128
// entries at a time, in two loads that do not wait for each other; longer lists take rounds of 64 before that.
template <class At>
static __device__ __forceinline__ DecodeReq find_request(At &&at, int n, int u, int *req) {
    const int l = threadIdx.x & 63;
    int lo = 0;
    while (n > 128) {
        const int step = (n + 63) / 64;
        const bool before = l * step < n && at(lo + l * step).slice0 <= u;
        const int k = __builtin_popcountll(__ballot(before)) - 1;
        lo += k * step;
        n = min(step, n - k * step);
    }
    const DecodeReq a = at(lo + min(l, n - 1)), b = at(lo + min(64 + l, n - 1));
    const int k = __builtin_popcountll(__ballot(l < n && a.slice0 <= u)) + __builtin_popcountll(__ballot(64 + l < n && b.slice0 <= u)) - 1;
    *req = lo + k;
    const int j = k & 63;
    auto pick = [&](int x, int y) { return k < 64 ? __builtin_amdgcn_readlane(x, j) : __builtin_amdgcn_readlane(y, j); };
    return DecodeReq{pick(a.ctx_len, b.ctx_len), pick(a.slice0, b.slice0), pick(a.part0, b.part0)};
}
#endif

#if defined(__HIP_DEVICE_COMPILE__)
// ARGUMENT: the list is `inl`, not in memory.  HEADS: the form of P V (as in attend below), -1 for the one that G calls for.
template <int D, bool FUSED, bool ARGUMENT, int HEADS>
static __device__ __forceinline__ void decode_slice(const DecodeParams &p, const DecodeList &inl, int G) {
    constexpr int ROWB = D * 2;            // bytes per K/V row
    constexpr int NJ = D / 32;             // MFMAs (and K loads) per page
    constexpr int E = D / 16;              // d-values of a V row per lane
    constexpr int PR = D + 4;              // floats of a head's row in LDS
    typedef typename VRow<D>::type vrow;

    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (all arguments in one trip, and with them the list if it is one of them)
    static_assert(DECODE_INLINE_REQS == 128, "two entries per lane");
    DecodeReq near, far;
    if constexpr (ARGUMENT) near = inl.r[l], far = inl.r[64 + l];
    asm volatile("" ::"s"(p.q), "s"(p.kv_pool), "s"(p.block_table), "s"(p.reqs), "s"(p.mirror_reqs), "s"(p.scratch), "s"(p.n_reqs),
                 "s"(p.slice_pages), "s"(p.Hq), "s"(p.Hkv), "s"(p.max_pages), "s"(p.num_pages), "s"(G));
    const int kvh = blockIdx.x % p.Hkv;
    const int slice = blockIdx.x / p.Hkv;
    int req;
    DecodeReq rq;
    if constexpr (ARGUMENT) {
        req = __builtin_popcountll(__ballot(l < p.n_reqs && near.slice0 <= slice)) +
              __builtin_popcountll(__ballot(64 + l < p.n_reqs && far.slice0 <= slice)) - 1;
        auto pick = [&](int x, int y) {                    // both read: no branch
            const int a = __builtin_amdgcn_readlane(x, req & 63), b = __builtin_amdgcn_readlane(y, req & 63);
            return req < 64 ? a : b;
        };
        rq = DecodeReq{pick(near.ctx_len, far.ctx_len), pick(near.slice0, far.slice0), pick(near.part0, far.part0)};
    } else {
        rq = find_request([&](int i) { return p.reqs[i]; }, p.n_reqs, slice, &req);
    }
    if (p.mirror_reqs != nullptr && kvh == 0 && slice == rq.slice0 && threadIdx.x == 0) p.mirror_reqs[req] = rq;
    const int pages = (rq.ctx_len + 15) >> 4;
    const int n_slices = pages > p.slice_pages ? (pages + p.slice_pages - 1) / p.slice_pages : 1;
    const int page0 = (slice - rq.slice0) * p.slice_pages, page1 = min(pages, page0 + p.slice_pages);
    const int g = l >> 4, c = l & 15;

    // this wave's pages: page0 + w, + 4, ...; their ids sit 64 at a time in one register
    const int32_t *bt = p.block_table + (int64_t)req * p.max_pages;
    const int n_mine = page1 - page0 > w ? (page1 - page0 - w + DEC_WAVES - 1) / DEC_WAVES : 0;
    auto load_ids = [&](int blk) {
        const int k = blk * 64 + l;
        int pg = k < n_mine ? bt[page0 + w + DEC_WAVES * k] : 0;
        return pg < 0 ? 0 : (pg >= p.num_pages ? p.num_pages - 1 : pg);
    };
    int ids = load_ids(0);

    // Q^T operand of step j: lane (g, c) holds q[head c][32j + 8g .. +7]; columns >= G are zero
    bf16x8 qB[NJ];
    {
        const __bf16 *qp = (const __bf16 *)p.q + ((int64_t)req * p.Hq + kvh * G + (c < G ? c : 0)) * D + 8 * g;
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            qB[j] = *(const bf16x8 *)(qp + 32 * j);
            if (c >= G) {
#pragma unroll
                for (int e = 0; e < 8; e++) qB[j][e] = (__bf16)0.f;
            }
        }
    }
    const float sc = 1.4426950408889634f * rsqrtf((float)D);   // scores in log2 units

    const int64_t page_bytes = 2 * (int64_t)p.Hkv * 16 * ROWB;
    const char *pool_k = (const char *)p.kv_pool + (int64_t)kvh * 16 * ROWB;
    const int64_t v_in_page = (int64_t)p.Hkv * 16 * ROWB;
    const int koff = c * ROWB + g * 16;                         // + 64 j
    const int voff = 4 * g * ROWB + c * 2 * E;                  // + i * ROWB

    struct PageRegs { bf16x8 k[NJ]; vrow v[4]; };
    auto load_page = [&](int k, PageRegs &r) {
        const char *kb = pool_k + (int64_t)__builtin_amdgcn_readlane(ids, k & 63) * page_bytes;
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            // K and V are read exactly once: streaming loads
            const u32x4 raw = __builtin_nontemporal_load((const u32x4 *)(kb + koff + 64 * j));
            __builtin_memcpy(&r.k[j], &raw, 16);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) r.v[i] = __builtin_nontemporal_load((const vrow *)(kb + v_in_page + voff + i * ROWB));
    };

    __shared__ __attribute__((aligned(16))) float part[DEC_WAVES][DEC_MAX_HEADS * PR];
    __shared__ float part_m[DEC_WAVES][DEC_MAX_HEADS], part_l[DEC_WAVES][DEC_MAX_HEADS];

    // The wave's pages, with P V on one of two instructions, and the wave's result to LDS.
    auto attend = [&](auto heads) __attribute__((always_inline)) {
        // HB: groups of four query heads on the 4x4x1 MFMA (1 up to 4 heads, 2 for 8), or 0: the 16 columns of the 16x16x4.
        constexpr int HB = decltype(heads)::value;
        // HB = 0: lane (g, c): acc[0][e][r] = O[d = E*(4g + r) + e][head c].  HB > 0: acc[hb][e][r] = this lane's share, the tokens of
        // its group g, of O[d = E*c + e][head 4 hb + r].  Reference and partial row sum of head c.
        constexpr int NB = HB > 0 ? HB : 1;
        f32x4 acc[NB][E];
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int e = 0; e < E; e++) acc[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        // (the lowest finite value, not -inf: keys whose scores are -inf count nothing against it, and the first score that
        // counts is still ahead of it by more than DEC_RESCALE_LOG2)
        float M = -__FLT_MAX__, lsum = 0.f;

        auto compute_page = [&](int k, PageRegs &r) {
            const int valid = rq.ctx_len - (page0 + w + DEC_WAVES * k) * 16;   // >= 1 tokens of this page count
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; j++) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r.k[j], qB[j], s, 0, 0, 0);
            // lane (g, c): s[i] = score of token 4g + i for head c
            float t[4];
#pragma unroll
            for (int i = 0; i < 4; i++) t[i] = 4 * g + i < valid ? fmaf(s[i], sc, -M) : -INFINITY;
            const float tm = fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]));
            if (__any(c < G && tm > DEC_RESCALE_LOG2)) {
                // move the reference of every head to the largest score the wave has seen
                float mx = -INFINITY;
#pragma unroll
                for (int i = 0; i < 4; i++) mx = fmaxf(mx, 4 * g + i < valid ? s[i] * sc : -INFINITY);
                mx = max_over_head(mx, 16);
                const float newM = fmaxf(M, mx);
                const float alpha = __builtin_amdgcn_exp2f(M - newM);      // 0 on the first page
                M = newM;
                lsum *= alpha;
#pragma unroll
                for (int i = 0; i < 4; i++) t[i] = 4 * g + i < valid ? fmaf(s[i], sc, -M) : -INFINITY;
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    float al[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) al[q] = HB > 0 ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), 4 * b + q)) : alpha;
#pragma unroll
                    for (int e = 0; e < E; e++)
#pragma unroll
                        for (int q = 0; q < 4; q++) acc[b][e][q] *= al[q];
                }
            }
            float pr[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                pr[i] = __builtin_amdgcn_exp2f(t[i]);
                lsum += pr[i];
            }
            if (valid < 16) {
                // rows past the context hold arbitrary pool bytes and must not reach the product
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (4 * g + i >= valid) r.v[i] = vrow{};
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int e = 0; e < E; e++) {
                    const unsigned u = r.v[i][e / 2];
                    const float v = __uint_as_float(e & 1 ? u & 0xffff0000u : u << 16);
                    // (operand A of HB > 0: block 4g + b of each group of four blocks, lanes 16 g + 4 b .., for all four of them)
                    if constexpr (HB == 0) acc[0][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, pr[i], acc[0][e], 0, 0, 0);
                    else acc[0][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(pr[i], v, acc[0][e], 2, 0, 0);
                    if constexpr (HB == 2) acc[1][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(pr[i], v, acc[1][e], 2, 1, 0);
                }
        };

        // the next page is in flight while one is being worked on
        PageRegs rg[2];
        if (n_mine > 0) load_page(0, rg[0]);
        for (int k0 = 0; k0 < n_mine; k0 += 2) {
#pragma unroll
            for (int b = 0; b < 2; b++) {
                const int k = k0 + b;
                if (k < n_mine) {
                    if (k + 1 < n_mine) {
                        if (((k + 1) & 63) == 0) ids = load_ids((k + 1) >> 6);
                        load_page(k + 1, rg[1 - b]);
                    }
                    compute_page(k, rg[b]);
                }
            }
        }
        lsum = fold16(lsum, lsum);
        lsum = fold32(lsum, lsum);

        // (rows padded by 16 bytes: the lanes of a 16-lane group store 16 bytes to a row each)
        if constexpr (HB == 0) {
            if (c < G) {
                float *ps = part[w] + c * PR + 4 * g * E;
#pragma unroll
                for (int q = 0; q < 4; q++)
#pragma unroll
                    for (int e = 0; e < E; e += 4) *(f32x4 *)(ps + q * E + e) = f32x4{acc[0][e][q], acc[0][e + 1][q], acc[0][e + 2][q], acc[0][e + 3][q]};
            }
        } else {
            // the four groups' shares: folded so that group g is left with head 4 b + g
#pragma unroll
            for (int b = 0; b < NB; b++) {
                float o[E];
#pragma unroll
                for (int e = 0; e < E; e++) o[e] = fold16(fold32(acc[b][e][0], acc[b][e][2]), fold32(acc[b][e][1], acc[b][e][3]));
                float *ps = part[w] + (4 * b + g) * PR + c * E;
#pragma unroll
                for (int e = 0; e < E; e += 4) *(f32x4 *)(ps + e) = f32x4{o[e], o[e + 1], o[e + 2], o[e + 3]};
            }
        }
        if (c < G && g == 0) {
            part_m[w][c] = M;
            part_l[w][c] = lsum;
        }
    };
    if constexpr (HEADS >= 0) attend(IntC<HEADS>{});
    else if (G <= 4) attend(IntC<1>{});
    else if (G == 8) attend(IntC<2>{});
    else attend(IntC<0>{});

    // the four waves of the work-group meet
    __syncthreads();
    const int PS = (G * (D + 2) + 3) & ~3;
    const int64_t stride = (int64_t)p.Hkv * PS;                        // between consecutive slices
    float *dst = p.scratch + ((int64_t)(rq.part0 + slice - rq.slice0) * p.Hkv + kvh) * PS;
    __bf16 *out = (__bf16 *)p.out + ((int64_t)req * p.Hq + kvh * G) * D;
    for (int it = threadIdx.x; it < G * D / 4; it += DEC_THREADS) {
        const int h = it * 4 / D, d = it * 4 % D;
        float Mx = -INFINITY, den = 0.f;
#pragma unroll
        for (int ww = 0; ww < DEC_WAVES; ww++) Mx = fmaxf(Mx, part_m[ww][h]);
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ww = 0; ww < DEC_WAVES; ww++) {
            const float f = weight(part_m[ww][h], Mx);
            const f32x4 x = *(const f32x4 *)(part[ww] + h * PR + d);
#pragma unroll
            for (int e = 0; e < 4; e++) num[e] = fmaf(f, x[e], num[e]);
            den = fmaf(f, part_l[ww][h], den);
        }
        if (n_slices == 1) {
            bf16x4 r;
#pragma unroll
            for (int e = 0; e < 4; e++) r[e] = (__bf16)(den > 0.f ? num[e] / den : 0.f);
            *(bf16x4 *)(out + it * 4) = r;
        } else {
            store_partial<FUSED>(dst + it * 4, num[0], num[1]);
            store_partial<FUSED>(dst + it * 4 + 2, num[2], num[3]);
            if (d == 0) store_partial<FUSED>(dst + G * D + 2 * h, Mx, den);
        }
    }
    if constexpr (FUSED) {
        if (n_slices == 1) return;
        // The last work-group to get here merges.  Every thread waits until its stores have been written through
        // to where the other XCDs see them before thread 0 counts the work-group in; the counter wraps to 0 for
        // the next launch on this stream.  What makes the partials visible is this chip and not the memory model: agent-scope
        // stores go past the XCD's L2, and once vmcnt says that they are done the count, which is made there too, comes
        // after them.  A release to the device would say the same portably, but writes the XCD's whole L2 back: with one per
        // work-group the full-size batch took 474 us and not 360.  The release to the work-group costs nothing here and keeps
        // the compiler from moving a store behind the wait.
        __shared__ int is_last;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0)
        __syncthreads();
        if (threadIdx.x == 0) {
            is_last = atomicInc(p.counters + (int64_t)req * p.Hkv + kvh, (unsigned)n_slices - 1) == (unsigned)n_slices - 1;
        }
        __syncthreads();
        if (!is_last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        // (the host takes this form only where the partials are within MERGE_HELD)
        merge_held<D>(p.scratch + ((int64_t)rq.part0 * p.Hkv + kvh) * PS, stride, n_slices, G, out);
    }
}
#endif

#define DECODE_KERNEL __global__ __launch_bounds__(DEC_THREADS) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 4, D == 128 ? 2 : 4)))

// Lists in memory: all head counts at d = 64, up to four heads at d = 128.
template <int D, bool FUSED>
DECODE_KERNEL void decode_bf16_kernel(DecodeParams p, DecodeList inl, int G) {
#if defined(__HIP_DEVICE_COMPILE__)
    decode_slice<D, FUSED, false, D == 128 ? 1 : -1>(p, inl, G);
#endif
}

// ... eight and sixteen heads of 128
template <int D, bool FUSED, int HEADS>
DECODE_KERNEL void decode_bf16_heads_kernel(DecodeParams p, DecodeList inl, int G) {
#if defined(__HIP_DEVICE_COMPILE__)
    decode_slice<D, FUSED, false, HEADS>(p, inl, G);
#endif
}

// the list as an argument
template <int D, bool FUSED, int HEADS>
DECODE_KERNEL void decode_bf16_list_kernel(DecodeParams p, DecodeList inl, int G) {
#if defined(__HIP_DEVICE_COMPILE__)
    decode_slice<D, FUSED, true, HEADS>(p, inl, G);
#endif
}

// Second kernel of the form that keeps no counters: work-groups = (request, KV head, chunk of the output).
template <int D>
__global__ __launch_bounds__(DEC_THREADS) void decode_merge_kernel(DecodeParams p, DecodeList inl, int G) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int chunks = max(1, G * D / 4 / MERGE_ITEMS), chunk = blockIdx.x % chunks;
    const int kvh = blockIdx.x / chunks % p.Hkv, req = blockIdx.x / chunks / p.Hkv;
    const DecodeReq rq = p.reqs != nullptr ? p.reqs[req] : inl.r[req];
    const int pages = (rq.ctx_len + 15) >> 4;
    if (pages <= p.slice_pages) return;                               // the first kernel wrote the row
    const int PS = (G * (D + 2) + 3) & ~3;
    const float *base = p.scratch + ((int64_t)rq.part0 * p.Hkv + kvh) * PS;
    const int64_t stride = (int64_t)p.Hkv * PS;
    const int n = (pages + p.slice_pages - 1) / p.slice_pages;
    __bf16 *out = (__bf16 *)p.out + ((int64_t)req * p.Hq + kvh * G) * D;
    if ((int64_t)n * (G * D / 4) > MERGE_HELD) merge_slices<D>(base, stride, n, G, chunk, out);
    else if (chunk == 0) merge_held<D>(base, stride, n, G, out);
#endif
}

__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t *w, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) w[i] = 0;
}

hipError_t launch_clear_words(uint32_t *w, int n, hipStream_t s) {
    hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, n);
    return hipGetLastError();
}

// At d = 128 every form of P V has kernels of its own: a wave without pages goes past the loads of Q, and one with pages asks for
// Q and its first page together, where with all forms behind a branch every wave waits for Q first.  us, one kernel for all heads -> its
// own: 129 x 8 tokens at 32/2 heads of 128 5.5 -> 4.7, 1000 x 8 20.0 -> 18.0, 400 x 8 at 32/8 22.1 -> 20.4, 400 x 300 80.7 and 80.7, 64 of 1024 .. 16384
// with append 357 -> 355.  At d = 64, where a page is half as long and Q comes with its ids, that loses: 24 of 17 .. 4097 at 16/2 with append
// 14.5 -> 15.1, 400 x 64 at 16/1 4.9 -> 5.3.  So it does at d = 128 where the list is an argument and a second kernel merges:
// static calls with append, its own and one kernel for all heads, 2 x 16033 tokens at 32/8 29.5, 28.8; 16 x 1000 20.2, 19.6; 4 x 4000 20.1, 19.5; 2 x 16033 at 32/2
// 20.3, 20.1; and the same in both within 0.2 %: 64 of 1024 .. 16384 and 128 x 1000.
template <int D, bool FUSED>
static void (*decode_kernel(const DecodeParams &p, int G))(DecodeParams, DecodeList, int) {
    const bool list = p.reqs == nullptr;
    if constexpr (D == 64) return list ? decode_bf16_list_kernel<D, FUSED, -1> : decode_bf16_kernel<D, FUSED>;
    else if (G <= 4) return list ? decode_bf16_list_kernel<D, FUSED, FUSED ? 1 : -1> : decode_bf16_kernel<D, FUSED>;
    else if (G == 8) return list ? decode_bf16_list_kernel<D, FUSED, FUSED ? 2 : -1> : decode_bf16_heads_kernel<D, FUSED, 2>;
    else return list ? decode_bf16_list_kernel<D, FUSED, FUSED ? 0 : -1> : decode_bf16_heads_kernel<D, FUSED, 0>;
}

template <int D>
static hipError_t launch_decode_one(const DecodeParams &p, const DecodeList &inl, int G, hipStream_t s) {
    const dim3 grid((unsigned)p.n_slices * p.Hkv);
    hipLaunchKernelGGL((p.counters != nullptr ? decode_kernel<D, true>(p, G) : decode_kernel<D, false>(p, G)), grid, dim3(DEC_THREADS), 0, s, p, inl, G);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.counters != nullptr || p.n_slices == p.n_reqs) return e;          // every request is one slice
    hipLaunchKernelGGL((decode_merge_kernel<D>), dim3((unsigned)p.n_reqs * p.Hkv * merge_chunks(D, G)), dim3(DEC_THREADS), 0, s, p, inl, G);
    return hipGetLastError();
}

hipError_t launch_decode_bf16(const DecodeParams &p, const DecodeList &inl, int head_dim, hipStream_t s) {
    const int G = p.Hq / p.Hkv;
    return head_dim == 128 ? launch_decode_one<128>(p, inl, G, s) : launch_decode_one<64>(p, inl, G, s);
}

}  // namespace pbkv
