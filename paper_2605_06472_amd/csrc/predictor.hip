// Forward pass of the workflow predictor (App. B) for gfx950.
//
// prepare (once per set of weights)
//   predictor_tables_kernel   H^(2) by the two GraphSAGE layers, the |V| x |V| table
//                             S[v][u] = (W_q H2[v]) . H2[u] / sqrt(d) of attention scores between
//                             agents: everything request-independent
//   predictor_split_kernel    W_t = hi + lo, two bf16 matrices (16 significand bits together), stored in
//                             the order the projection's MFMA operands are read, and the head's weights in the
//                             order of the head's
// forward (per batch)
//   predictor_project_kernel  W_t x on the matrix cores: work-group = 32 requests x one slice of
//                             d_x, operands straight from global memory into the MFMA registers
//                             (x is row-major along d_x, which is the MFMA's k direction), the waves
//                             split the slice, partial sums to the workspace
//   predictor_head_kernel     four or eight requests per work-group: h_txt = ReLU(sum of the slices), h_cur,
//                             the history attention by table look-up, the two head layers on the fp32 matrix
//                             cores, K softmaxes
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

#include "../../include/pbkv.h"
#include "../../include/pbkv_predictor.h"
#include "pbkv_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int KS_MAX = 16;          // most slices of d_x a batch is split into
constexpr int TARGET_WGS = 256;     // projection work-groups aimed for (one per CU)

int64_t align256(int64_t v) { return (v + 255) & ~(int64_t)255; }

// Workspace layout (byte offsets, each 256-byte aligned).
struct Layout {
    int64_t h2, s, wat, ba, wbt, bb, ah1, h1, ah2, q, wp, partial, total;
    int bpad;
};

Layout layout(const pbkv_predictor_shape *p, int32_t max_batch) {
    const int64_t V = p->num_agents, d = p->d, hid = p->hidden, kv1 = (int64_t)p->horizon * (V + 1);
    Layout L;
    int64_t o = 0;
    auto take = [&](int64_t bytes) { int64_t at = o; o = align256(o + bytes); return at; };
    L.h2 = take(V * d * 4);
    L.s = take(V * V * 4);
    L.wat = take(3 * d * hid * 4);
    L.ba = take(hid * 4);
    L.bb = take(kv1 * 4);
    // (the padding of its last group of four hidden units, up to 3 kv1 <= 24 (|V| + 1) floats, stands in the intermediates behind
    // it, which are dead when it is written: ah1, h1 and ah2 are 96 |V| floats or more)
    L.wbt = take(hid * kv1 * 4);
    L.ah1 = take(V * d * 4);      // intermediates of the table kernel, each written once
    L.h1 = take(V * d * 4);
    L.ah2 = take(V * d * 4);
    L.q = take(V * d * 4);
    L.wp = take(2 * d * (int64_t)p->d_x * 2);      // W_t as hi + lo bf16 in operand order
    L.bpad = (max_batch + 31) / 32 * 32;
    L.partial = take((int64_t)KS_MAX * L.bpad * d * 4);
    L.total = o;
    return L;
}

int check_shape(const pbkv_predictor_shape *p) {
    if (!p) return pbkv::set_error(PBKV_ERR_NULL, "predictor shape is NULL");
    if (p->num_agents < 1 || p->num_agents > 64) return pbkv::set_error(PBKV_ERR_SHAPE, "num_agents %d not in [1, 64]", p->num_agents);
    if (p->d != 32 && p->d != 64 && p->d != 128) return pbkv::set_error(PBKV_ERR_SHAPE, "d %d is not 32, 64 or 128", p->d);
    if (p->d_x < 64 || p->d_x % 16) return pbkv::set_error(PBKV_ERR_SHAPE, "d_x %d is not a multiple of 16 >= 64", p->d_x);
    if (p->hidden < 1 || p->hidden > 256) return pbkv::set_error(PBKV_ERR_SHAPE, "hidden %d not in [1, 256]", p->hidden);
    if (p->horizon < 1 || p->horizon > 8) return pbkv::set_error(PBKV_ERR_SHAPE, "horizon %d not in [1, 8]", p->horizon);
    if (p->max_prefix < 0 || p->max_prefix > 64) return pbkv::set_error(PBKV_ERR_SHAPE, "max_prefix %d not in [0, 64]", p->max_prefix);
    return PBKV_OK;
}

int check_dev(const void *ptr, const char *name, int align) {
    if (!ptr) return pbkv::set_error(PBKV_ERR_NULL, "%s is NULL", name);
    if ((uintptr_t)ptr & (uintptr_t)(align - 1)) return pbkv::set_error(PBKV_ERR_SHAPE, "%s is not %d-byte aligned", name, align);
    hipPointerAttribute_t a;
    hipError_t e = hipPointerGetAttributes(&a, ptr);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return pbkv::set_error(PBKV_ERR_DEVICE, "%s: not a device pointer (%s)", name, hipGetErrorString(e));
    }
    if (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged)
        return pbkv::set_error(PBKV_ERR_DEVICE, "%s: expected device memory", name);
    return PBKV_OK;
}

struct TablesParams {
    const float *emb, *trans, *w1, *w2, *wq;
    float *h2, *s, *ah1, *h1, *ah2, *q;
    int V, d;
};

// The head's weights as the forward pass reads them (behind the tables kernel, whose intermediates wbt may reach into).
struct HeadWeights {
    const float *wa, *ba, *wb, *bb;
    float *wat, *ba_out, *wbt, *bb_out;
    int hidden, kv1;
};

// One work-group.  Phases are separated by barriers; every intermediate array is written in one
// phase and only read in later ones.
__global__ __launch_bounds__(256) void predictor_tables_kernel(TablesParams p) {
    const int t = threadIdx.x, V = p.V, d = p.d;
    // A H for a [V][d] matrix H
    auto propagate = [&](const float *H, float *AH) {
        for (int e = t; e < V * d; e += 256) {
            const int v = e / d, f = e % d;
            float acc = 0.f;
            for (int u = 0; u < V; u++) acc = fmaf(p.trans[v * V + u], H[u * d + f], acc);
            AH[e] = acc;
        }
    };
    // ReLU([H || AH] W^T), W [d][2d]   (GraphSAGE equation, App. B)
    auto layer = [&](const float *H, const float *AH, const float *Wm, float *out) {
        for (int e = t; e < V * d; e += 256) {
            const int v = e / d, g = e % d;
            float acc = 0.f;
            for (int c = 0; c < d; c++) acc = fmaf(Wm[g * 2 * d + c], H[v * d + c], acc);
            for (int c = 0; c < d; c++) acc = fmaf(Wm[g * 2 * d + d + c], AH[v * d + c], acc);
            out[e] = fmaxf(acc, 0.f);
        }
    };
    propagate(p.emb, p.ah1);
    __syncthreads();
    layer(p.emb, p.ah1, p.w1, p.h1);
    __syncthreads();
    propagate(p.h1, p.ah2);
    __syncthreads();
    layer(p.h1, p.ah2, p.w2, p.h2);
    __syncthreads();
    // queries W_q H2[v] of every agent (history-attention equation, App. B)
    for (int e = t; e < V * d; e += 256) {
        const int v = e / d, g = e % d;
        float acc = 0.f;
        for (int c = 0; c < d; c++) acc = fmaf(p.wq[g * d + c], p.h2[v * d + c], acc);
        p.q[e] = acc;
    }
    __syncthreads();
    const float inv_sqrt_d = 1.0f / sqrtf((float)d);
    for (int e = t; e < V * V; e += 256) {
        const int v = e / V, u = e % V;
        float acc = 0.f;
        for (int g = 0; g < d; g++) acc = fmaf(p.q[v * d + g], p.h2[u * d + g], acc);
        p.s[e] = acc * inv_sqrt_d;
    }
}

// W_t in the order the projection reads it.  w = hi + lo with hi = bf16(w), lo = bf16(w - hi): the
// sum is w to 2^-17 relative.  For k-step s (16 columns of d_x) and feature block cb (32 rows) the
// 64 lanes' hi operands are 1 KiB contiguous, then the 64 lo operands:
//   wp[(((s * DB + cb) * 2 + part) * 64 + lane) * 8 + e] = part(W_t[32 cb + lane % 32][16 s + 8 (lane / 32) + e])
__global__ __launch_bounds__(256) void predictor_split_kernel(const float *w, __bf16 *wp, int d, int d_x, HeadWeights h) {
    const int DB = d / 32, ksteps = d_x / 16;
    const int64_t n = (int64_t)ksteps * DB * 64;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int lane = (int)(i % 64), cb = (int)(i / 64 % DB), st = (int)(i / 64 / DB);
        const float *src = w + (int64_t)(32 * cb + lane % 32) * d_x + 16 * st + 8 * (lane / 32);
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float v = src[e];
            hi[e] = (__bf16)v;
            lo[e] = (__bf16)(v - (float)hi[e]);
        }
        bf16x8 *dst = (bf16x8 *)wp + ((int64_t)(st * DB + cb) * 2) * 64 + lane;
        dst[0] = hi;
        dst[64] = lo;
    }
    // head weights, [inputs / 4][output][4 inputs]: a lane reads four inputs of its output, a wave contiguous memory
    const int t0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    for (int e = t0; e < 3 * d * h.hidden; e += step) {
        const int j = e / 4 % h.hidden, k = e / 4 / h.hidden * 4 + e % 4;
        h.wat[e] = h.wa[j * 3 * d + k];
    }
    for (int e = t0; e < (h.hidden + 3) / 4 * 4 * h.kv1; e += step) {
        const int o = e / 4 % h.kv1, j = e / 4 / h.kv1 * 4 + e % 4;
        h.wbt[e] = j < h.hidden ? h.wb[o * h.hidden + j] : 0.f;
    }
    for (int e = t0; e < h.hidden; e += step) h.ba_out[e] = h.ba[e];
    for (int e = t0; e < h.kv1; e += step) h.bb_out[e] = h.bb[e];
}

struct ProjectParams {
    const __bf16 *x, *wp;
    float *partial;
    int batch, bpad, d_x, steps_per_slice, ksteps;
};

// Work-group (rb, slice): requests 32*rb .. +31, k-steps [slice*sps, (slice+1)*sps) of 16 columns
// of d_x each, handed to the waves in groups of a few consecutive k-steps.  out^T = W_t x^T: the A operand is a 32 x 16 block of W_t (rows = features), read
// from the prepared operand-order copy (1 KiB contiguous per wave load); the B operand is a 16 x 32
// block of x^T (columns = requests): lane (i = l%32, h = l/32) holds the 8 consecutive d_x entries
// 8h .. 8h+7 of row i, one 16-byte load from the row-major x.  The kernel is bound by memory
// latency, so a wave issues all loads of a group before its first MFMA.
template <int DB, int NW>     // d / 32, waves per work-group
__global__ __launch_bounds__(64 * NW) void predictor_project_kernel(ProjectParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int D = 32 * DB;
    constexpr int CH = DB == 4 ? 3 : 5;                   // consecutive k-steps per group: all their operands are held at once
    __shared__ float red[NW / 2][32][D + 4];
    const int l = threadIdx.x & 63, li = l & 31, lh = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rb = blockIdx.x, slice = blockIdx.y;
    const int s0 = slice * p.steps_per_slice;
    const int s1 = min(s0 + p.steps_per_slice, p.ksteps);
    const int row = rb * 32 + li;
    const bool valid = row < p.batch;
    const __bf16 *xp = p.x + (int64_t)(valid ? row : 0) * p.d_x + 8 * lh;
    const bf16x8 *wp = (const bf16x8 *)p.wp + l;
    f32x16 acc[DB];
#pragma unroll
    for (int cb = 0; cb < DB; cb++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[cb][r] = 0.f;
    bf16x8 zero;
#pragma unroll
    for (int e = 0; e < 8; e++) zero[e] = (__bf16)0.f;
    for (int base = s0 + CH * w; base < s1; base += CH * NW) {
        bf16x8 xo[CH], ho[CH][DB], lo[CH][DB];
#pragma unroll
        for (int c = 0; c < CH; c++) {
            const int sc = base + c < s1 ? base + c : base;   // past the slice: a valid address, operand zeroed below
            xo[c] = *(const bf16x8 *)(xp + sc * 16);
#pragma unroll
            for (int cb = 0; cb < DB; cb++) {
                ho[c][cb] = wp[((int64_t)(sc * DB + cb) * 2) * 64];
                lo[c][cb] = wp[((int64_t)(sc * DB + cb) * 2 + 1) * 64];
            }
        }
#pragma unroll
        for (int c = 0; c < CH; c++) {
            const bool on = valid && base + c < s1;
            const bf16x8 xb = on ? xo[c] : zero;
#pragma unroll
            for (int cb = 0; cb < DB; cb++) {
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ho[c][cb], xb, acc[cb], 0, 0, 0);
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo[c][cb], xb, acc[cb], 0, 0, 0);
            }
        }
    }
    // The waves' sums meet in LDS: the upper half hands over, the lower half adds and hands over, then every
    // thread sums what is left of one run of four features: two exchanges, where a binary tree has a store, a
    // load and two barriers per level and leaves a shrinking part of the waves at work (9500 -> 8900 clocks for
    // the kernel at d = 64; the rest is W_t's way into registers).  The order of the additions is that of the tree.
    // Register r of lane (li, lh) is feature 32*cb + 8*(r/4) + 4*lh + r%4 of request li.
    constexpr int HALF = NW / 2;
    auto exchange = [&](bool store) {
        float *at = &red[w & (HALF - 1)][li][4 * lh];
#pragma unroll
        for (int cb = 0; cb < DB; cb++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                f32x4 *slot = (f32x4 *)(at + 32 * cb + 8 * g);
                f32x4 v;
#pragma unroll
                for (int c = 0; c < 4; c++) v[c] = acc[cb][4 * g + c];
                *slot = store ? v : v + *slot;
            }
    };
    if (w >= HALF) exchange(true);
    __syncthreads();
    if (w < HALF) exchange(false);
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * D / 4; i += 64 * NW) {
        const int r = i / (D / 4), f = 4 * (i % (D / 4));
        f32x4 v[HALF];
#pragma unroll
        for (int k = 0; k < HALF; k++) v[k] = *(const f32x4 *)&red[k][r][f];
#pragma unroll
        for (int half = HALF / 2; half >= 1; half >>= 1)
#pragma unroll
            for (int k = 0; k < half; k++) v[k] += v[k + half];
        *(f32x4 *)(p.partial + ((int64_t)slice * p.bpad + rb * 32 + r) * D + f) = v[0];
    }
#endif
}

constexpr int HEAD_WAVES = 8;
constexpr int HNT = 64 * HEAD_WAVES;    // threads of a head work-group

// A layer's outputs are taken 64 at a time (one per lane), its inputs are dealt out to as many parts as leave every
// wave one (outputs, part) item, or one part where the outputs alone are more than that.
struct HeadLayer {
    int outputs, groups;                // groups of four inputs
    int chunks, parts, pitch;
    int per_part, inv_chunks;           // groups of a part; x / chunks is x inv_chunks / 2^16 (x < 64)
};
HeadLayer head_layer(int inputs, int outputs) {
    HeadLayer y;
    y.outputs = outputs;
    y.groups = (inputs + 3) / 4;
    y.chunks = (outputs + 63) / 64;
    y.parts = y.chunks < HEAD_WAVES ? HEAD_WAVES / y.chunks : 1;
    y.pitch = 64 * y.chunks + 16;       // floats between requests of a part's sums: four requests' 16-byte stores meet no bank twice
    y.per_part = (y.groups + y.parts - 1) / y.parts;
    y.inv_chunks = 65536 / y.chunks + 1;
    return y;
}

// LDS of the head kernel, in floats (dynamic: it grows with |V| d and exceeds 64 KiB for the largest shapes).
struct HeadLds {
    int z, hid, red, h2, s, ba, bb, total;
    int zp, hp;                         // pitches of z and hid: 16 bytes past a multiple of their rows, for the same reason
};
HeadLds head_lds(int RPB, int V, int d, int hidden, int kv1, const HeadLayer &y1, const HeadLayer &y2) {
    HeadLds o;
    int at = 0;
    auto take = [&](int n) { int r = at; at += (n + 3) & ~3; return r; };
    const int r1 = y1.parts * y1.pitch, r2 = y2.parts * y2.pitch;
    o.zp = 3 * d + 4;
    o.hp = ((hidden + 3) & ~3) + 4;
    o.z = take(RPB * o.zp);
    o.hid = take(RPB * o.hp);
    o.red = take(RPB * (r1 > r2 ? r1 : r2));
    o.h2 = take(V * d);
    o.s = take(V * V);
    o.ba = take(hidden);
    o.bb = take(kv1);
    o.total = at;
    return o;
}

struct HeadParams {
    const float *partial, *h2, *s, *wat, *ba, *wbt, *bb;
    const int32_t *cur_agent, *prefix, *prefix_len;
    float *probs;
    int64_t slice_floats;               // between a request's slices of the projection
    int batch, n_slices, V, d, hidden, K, L, kv1;
    int inv_K;                          // row / K is row inv_K / 2^16 (row < 64)
    HeadLds o;
    HeadLayer y1, y2;
};

// Up to this many requests the head takes four per work-group (one work-group per CU), above eight (every work-group
// reads all tables and weights).  us per pass with four and with eight: batch 1 10.0 and 10.9, 1024 12.3 and 13.8, 1536 17.9 and 16.8,
// 4096 31.2 and 27.2; 32 agents, d = 128, hidden = 256, horizon 4: 1024 27.4 and 34.0, 2048 37.8 and 40.3, 4096 63.9 and 57.0.
constexpr int HEAD_SMALL_BATCH = 1024;

#if defined(__HIP_DEVICE_COMPILE__)
// Over a row of 16 lanes, in every lane of it (rotations: the lanes get the same bits).
template <int CTRL> static __device__ __forceinline__ float row_ror(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
static __device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, row_ror<0x128>(v));
    v = fmaxf(v, row_ror<0x124>(v));
    v = fmaxf(v, row_ror<0x122>(v));
    return fmaxf(v, row_ror<0x121>(v));
}
static __device__ __forceinline__ float row_sum(float v) {
    v += row_ror<0x128>(v);
    v += row_ror<0x124>(v);
    v += row_ror<0x122>(v);
    return v + row_ror<0x121>(v);
}
// ... and over the whole wave; lanes n and up hold the neutral value, so up to 16 one row will do (its lanes get the result).
static __device__ __forceinline__ float wave_max(float v, int n) {
    v = row_max(v);
    if (n > 16) {
        v = fmaxf(v, __shfl_xor(v, 16, 64));
        v = fmaxf(v, __shfl_xor(v, 32, 64));
    }
    return v;
}
static __device__ __forceinline__ float wave_sum(float v, int n) {
    v = row_sum(v);
    if (n > 16) {
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
    }
    return v;
}
#endif

// Work-group = RPB requests, eight waves.  The work per request is tiny (10 k multiply-adds at the sizes of the header);
// what the kernel costs is one cold round trip to memory, the issue of its instructions and a chain of
// dependent phases.  Hence:
//   * both layers on the 4x4x1 fp32 MFMA (16 blocks): a lane is one output, the four columns are four requests, so
//     one instruction is 64 outputs x 4 requests of one input, in fp32 throughout, and a weight is read
//     by one wave, once, from global memory straight into the operand register (the prepared copies hold four
//     consecutive inputs of an output in 16 bytes, 1 KiB contiguous per wave load).  No weight passes through LDS;
//   * everything that does not depend on another load -- the slices of the projection, the indices, the tables, the
//     first weights of both layers -- is asked for before the first use;
//   * a request's attention over its prefix stays in one wave (row rotations, lane reads): no barrier inside it;
//   * a softmax belongs to 16 lanes, which also add the parts of their logits.
// 1024 states of 8 agents, d = hidden = 64, horizon 3: 14.4 us per pass over an x that stays in the caches, now 11.6 (4096 states
// 35 -> 26, one 12.4 -> 9.3); 32 agents, d = 128, hidden = 256, horizon 4: 1024 states 49.8 -> 25.7, 4096 138 -> 64.  (Before, W_a and
// W_b went through LDS and the layers ran on the vector ALU: of the 8.5 us of a work-group 2.6 went to the two layers, 1.7 to the stores of
// the staged weights and the barrier behind them; at the wide model 36 of 42 to the layers.)
// A request past the end of the batch is computed as request batch-1 again and stores nothing, so
// that all threads walk the same barriers.
template <int RPB>     // requests per work-group: 4 or 8
__global__ __launch_bounds__(HNT) void predictor_head_kernel(HeadParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int RT = RPB / 4, WPR = HEAD_WAVES / RPB;   // requests / 4, waves per request
    const int t = threadIdx.x, l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int b0 = blockIdx.x * RPB;
    const int V = p.V, d = p.d, hidden = p.hidden, V1 = p.V + 1, kv1 = p.kv1;
    const HeadLds &o = p.o;
    float *z = lds + o.z, *hid = lds + o.hid, *red = lds + o.red;
    // (all arguments in one trip: the compiler would fetch them as it comes to them)
    asm volatile("" ::"s"(p.partial), "s"(p.h2), "s"(p.s), "s"(p.wat), "s"(p.ba), "s"(p.wbt), "s"(p.bb), "s"(p.cur_agent), "s"(p.prefix),
                 "s"(p.prefix_len), "s"(p.batch), "s"(p.slice_floats), "s"(p.n_slices), "s"(p.L), "s"(p.y1.chunks), "s"(p.y2.chunks));

    // ---- every load that waits for no other ------------------------------------------------------
    const int r = w % RPB, req = min(b0 + r, p.batch - 1);            // the wave's request
    const int nf = d / WPR, f0 = (w / RPB) * nf;                      // ... and its features of it
    const int cur_len = (l & 1 ? p.prefix_len : p.cur_agent)[req];    // (per lane: nothing waits for it here)
    int pre = 0;
    if (l < p.L) pre = p.prefix[(int64_t)req * p.L + l];
    constexpr int NF = RPB == 4 ? 1 : 2;                              // features per lane, at most
    static_assert(KS_MAX == 16, "two runs of eight slices");
    float part[NF][KS_MAX];
#pragma unroll
    for (int q = 0; q < NF; q++) {
        const float *src = p.partial + (int64_t)req * d + f0 + min(l + 64 * q, nf - 1);
        auto slices = [&](int first) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 8; k++) part[q][first + k] = src[min(first + k, p.n_slices - 1) * p.slice_floats];
        };
#pragma unroll
        for (int sl = 8; sl < KS_MAX; sl++) part[q][sl] = 0.f;
        if (64 * q < nf) {                                            // (uniform, and so is the next)
            slices(0);
            if (p.n_slices > 8) slices(8);
        }
    }
    // a layer's item: `chunk` (64 outputs), part `part` of the groups of four inputs
    struct Item { const f32x4 *wt; int chunk, part, g0, g1; };
    auto item = [&](const HeadLayer &y, const float *wt, int i) {
        Item it;
        it.part = i * y.inv_chunks >> 16;
        it.chunk = i - it.part * y.chunks;
        it.g0 = min(it.part * y.per_part, y.groups);
        it.g1 = min(it.g0 + y.per_part, y.groups);
        it.wt = (const f32x4 *)wt + min(it.chunk * 64 + l, y.outputs - 1);       // + group * outputs
        return it;
    };
    constexpr int PW1 = 6, PW2 = 2;                       // groups whose weights are asked for here
    const Item i1 = item(p.y1, p.wat, w), i2 = item(p.y2, p.wbt, w);
    const bool has1 = w < p.y1.chunks * p.y1.parts, has2 = w < p.y2.chunks * p.y2.parts;
    f32x4 w1[PW1], w2[PW2];
#pragma unroll
    for (int k = 0; k < PW1; k++) w1[k] = i1.wt[min(i1.g0 + k, p.y1.groups - 1) * hidden];
#pragma unroll
    for (int k = 0; k < PW2; k++) w2[k] = i2.wt[min(i2.g0 + k, p.y2.groups - 1) * kv1];
    // the tables (their places in the workspace are padded to 256 bytes, those in LDS to 16); what is left of large ones follows below
    const int h4 = V * d / 4, s4 = (V * V + 3) / 4;
    const f32x4 th = ((const f32x4 *)p.h2)[min(t, h4 - 1)], ts = ((const f32x4 *)p.s)[min(t, s4 - 1)];
    const float vba = p.ba[min(t, hidden - 1)], vbb0 = p.bb[min(t, kv1 - 1)], vbb1 = p.bb[min(t + HNT, kv1 - 1)];

    int cur = __builtin_amdgcn_readlane(cur_len, 0), len = __builtin_amdgcn_readlane(cur_len, 1);
    cur = cur < 0 ? 0 : (cur >= V ? V - 1 : cur);
    len = len < 0 ? 0 : (len > p.L ? p.L : len);
    pre = pre < 0 ? 0 : (pre >= V ? V - 1 : pre);
    f32x4 *lh2 = (f32x4 *)(lds + o.h2), *ls = (f32x4 *)(lds + o.s);
    if (t < h4) lh2[t] = th;
    if (t < s4) ls[t] = ts;
#pragma unroll 2
    for (int e = t + HNT; e < h4; e += HNT) lh2[e] = ((const f32x4 *)p.h2)[e];
    for (int e = t + HNT; e < s4; e += HNT) ls[e] = ((const f32x4 *)p.s)[e];
    if (t < hidden) lds[o.ba + t] = vba;
    if (t < kv1) lds[o.bb + t] = vbb0;
    if (t + HNT < kv1) lds[o.bb + t + HNT] = vbb1;
#pragma unroll
    for (int q = 0; q < NF; q++) {
        float acc = 0.f;
#pragma unroll
        for (int sl = 0; sl < KS_MAX; sl++) acc += sl < p.n_slices ? part[q][sl] : 0.f;
        if (l + 64 * q < nf) z[r * o.zp + 2 * d + f0 + l + 64 * q] = fmaxf(acc, 0.f);         // h_txt = ReLU(W_t x)
    }
    __syncthreads();

    // ---- (i) h_cur = H2[v_t]; (ii) attention over the prefix agents, lane i = position i -----------------
    {
        const float *h2 = lds + o.h2 + f0 + min(l, nf - 1);
        const float sc = l < len ? lds[o.s + cur * V + pre] : -INFINITY;
        const float mx = wave_max(sc, p.L);
        const float e = l < len ? expf(sc - mx) : 0.f;
        const float den = wave_sum(e, p.L);
        const float alpha = l < len ? e / den : 0.f;
        float acc[NF];
#pragma unroll
        for (int q = 0; q < NF; q++) acc[q] = 0.f;
        const int step = nf > 64 ? 64 : 0;                            // to a lane's second feature
        for (int i = 0; i < len; i += 4) {                            // (positions past the prefix weigh 0)
            float al[4], v[4][NF];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int ag = __builtin_amdgcn_readlane(pre, i + k);
                al[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), i + k));
#pragma unroll
                for (int q = 0; q < NF; q++) v[k][q] = h2[ag * d + q * step];
            }
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int q = 0; q < NF; q++) acc[q] = fmaf(al[k], v[k][q], acc[q]);
        }
        float *zr = z + r * o.zp + f0 + l;
#pragma unroll
        for (int q = 0; q < NF; q++)
            if (l + 64 * q < nf) {
                zr[64 * q] = h2[cur * d + q * step];
                zr[d + 64 * q] = acc[q];
            }
    }
    __syncthreads();

    // ---- a layer: out[request][output] = sum over inputs in[request][input] W[output][input], parts to `red`
    auto multiply = [&](const HeadLayer &y, const Item &it, const float *in, int pitch, const auto &first) __attribute__((always_inline)) {
        constexpr int PW = sizeof(first) / sizeof(f32x4), AHEAD = 8;
        f32x4 acc[RT];
#pragma unroll
        for (int q = 0; q < RT; q++) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        const float *row = in + (l & 3) * pitch;
        auto group = [&](const f32x4 &a, int g) __attribute__((always_inline)) {
            f32x4 b[RT];
#pragma unroll
            for (int q = 0; q < RT; q++) b[q] = *(const f32x4 *)&row[4 * q * pitch + 4 * g];
#pragma unroll
            for (int c = 0; c < 4; c++)
#pragma unroll
                for (int q = 0; q < RT; q++) acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[c], b[q][c], acc[q], 0, 0, 0);
        };
        f32x4 next[AHEAD];
        auto fetch = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < AHEAD; k++) next[k] = it.wt[min(g + k, it.g1 - 1) * y.outputs];
        };
        if (it.g0 + PW < it.g1) fetch(it.g0 + PW);
#pragma unroll
        for (int k = 0; k < PW; k++)
            if (it.g0 + k < it.g1) group(first[k], it.g0 + k);
        for (int g = it.g0 + PW; g < it.g1; g += AHEAD) {
            f32x4 a[AHEAD];
#pragma unroll
            for (int k = 0; k < AHEAD; k++) a[k] = next[k];
            if (g + AHEAD < it.g1) fetch(g + AHEAD);
            if (g + AHEAD <= it.g1) {
#pragma unroll
                for (int k = 0; k < AHEAD; k++) group(a[k], g + k);
            } else {
#pragma unroll
                for (int k = 0; k < AHEAD; k++)
                    if (g + k < it.g1) group(a[k], g + k);
            }
        }
        // lane l: outputs 4 (l / 4) .. + 3 of its 64, request l % 4
#pragma unroll
        for (int q = 0; q < RT; q++)
            *(f32x4 *)&red[(it.part * RPB + 4 * q + (l & 3)) * y.pitch + it.chunk * 64 + (l & ~3)] = acc[q];
    };
    // the sum of a (request, output)'s parts, of which there are up to eight: all read at once
    auto parts_of = [&](const HeadLayer &y, int rr, int out) __attribute__((always_inline)) {
        const float *at = red + rr * y.pitch + out;
        float v[HEAD_WAVES], sum = 0.f;
#pragma unroll
        for (int k = 0; k < HEAD_WAVES; k++) v[k] = at[min(k, y.parts - 1) * RPB * y.pitch];
#pragma unroll
        for (int k = 0; k < HEAD_WAVES; k++) sum += k < y.parts ? v[k] : 0.f;
        return sum;
    };
    if (has1) multiply(p.y1, i1, z, o.zp, w1);
    __syncthreads();
    for (int j = (w / RPB) * 64 + l; j < 4 * p.y2.groups; j += 64 * WPR)              // (inputs past the last one count nothing)
        hid[r * o.hp + j] = j < hidden ? fmaxf(parts_of(p.y1, r, j) + lds[o.ba + j], 0.f) : 0.f;
    __syncthreads();
    if (has2) multiply(p.y2, i2, hid, o.hp, w2);
    for (int i = w + HEAD_WAVES; i < p.y2.chunks * p.y2.parts; i += HEAD_WAVES) {     // more than 512 outputs
        const Item it = item(p.y2, p.wbt, i);
        const f32x4 first[1] = {it.wt[0]};
        multiply(p.y2, it, hid, o.hp, first);
    }
    __syncthreads();

    // ---- one softmax per (request, step) over the |V| agents and END: 16 lanes, up to five values each ------
    const int c = t & 15, n_rows = min(RPB, p.batch - b0) * p.K;
    for (int row = t >> 4; row < n_rows; row += HNT / 16) {
        const int rr = row * p.inv_K >> 16, at = (row - rr * p.K) * V1;
        float v[5], mx = -INFINITY, sum = 0.f;
#pragma unroll
        for (int q = 0; q < 5; q++) {
            v[q] = -INFINITY;
            if (16 * q < V1 && c + 16 * q < V1) {
                v[q] = lds[o.bb + at + c + 16 * q] + parts_of(p.y2, rr, at + c + 16 * q);
                mx = fmaxf(mx, v[q]);
            }
        }
        mx = row_max(mx);
#pragma unroll
        for (int q = 0; q < 5; q++)
            if (16 * q < V1) {
                v[q] = c + 16 * q < V1 ? expf(v[q] - mx) : 0.f;
                sum += v[q];
            }
        sum = row_sum(sum);
#pragma unroll
        for (int q = 0; q < 5; q++)
            if (c + 16 * q < V1) p.probs[(int64_t)b0 * kv1 + row * V1 + c + 16 * q] = v[q] / sum;
    }
#endif
}

}  // namespace

extern "C" {

int64_t pbkv_predictor_workspace_bytes(const pbkv_predictor_shape *shape, int32_t max_batch) {
    pbkv::clear_error();
    if (check_shape(shape) != PBKV_OK) return 0;
    if (max_batch < 1) {
        pbkv::set_error(PBKV_ERR_RANGE, "max_batch %d is not positive", max_batch);
        return 0;
    }
    return layout(shape, max_batch).total;
}

int pbkv_predictor_prepare(const pbkv_predictor_shape *shape, const pbkv_predictor_weights *wts,
                           void *workspace, int64_t workspace_bytes, int32_t max_batch, void *stream) {
    pbkv::clear_error();
    if (int rc = check_shape(shape)) return rc;
    if (!wts) return pbkv::set_error(PBKV_ERR_NULL, "weights is NULL");
    if (max_batch < 1) return pbkv::set_error(PBKV_ERR_RANGE, "max_batch %d is not positive", max_batch);
    const Layout L = layout(shape, max_batch);
    if (workspace_bytes < L.total)
        return pbkv::set_error(PBKV_ERR_RANGE, "workspace of %lld bytes, %lld needed", (long long)workspace_bytes, (long long)L.total);
    if (int rc = check_dev(workspace, "workspace", 256)) return rc;
    const struct { const float *p; const char *n; } ptrs[] = {
        {wts->emb, "emb"}, {wts->trans, "trans"}, {wts->w1, "w1"}, {wts->w2, "w2"}, {wts->wq, "wq"},
        {wts->wt, "wt"}, {wts->wa, "wa"}, {wts->ba, "ba"}, {wts->wb, "wb"}, {wts->bb, "bb"}};
    for (const auto &e : ptrs)
        if (int rc = check_dev(e.p, e.n, 16)) return rc;
    char *ws = (char *)workspace;
    hipStream_t s = (hipStream_t)stream;
    TablesParams t;
    t.emb = wts->emb; t.trans = wts->trans; t.w1 = wts->w1; t.w2 = wts->w2; t.wq = wts->wq;
    t.h2 = (float *)(ws + L.h2); t.s = (float *)(ws + L.s);
    t.ah1 = (float *)(ws + L.ah1); t.h1 = (float *)(ws + L.h1); t.ah2 = (float *)(ws + L.ah2); t.q = (float *)(ws + L.q);
    t.V = shape->num_agents; t.d = shape->d;
    hipLaunchKernelGGL(predictor_tables_kernel, dim3(1), dim3(256), 0, s, t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return pbkv::set_error(PBKV_ERR_DEVICE, "predictor tables launch: %s", hipGetErrorString(e));
    const int64_t n = (int64_t)(shape->d_x / 16) * (shape->d / 32) * 64;
    const unsigned grid = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    HeadWeights h;
    h.wa = wts->wa; h.ba = wts->ba; h.wb = wts->wb; h.bb = wts->bb;
    h.wat = (float *)(ws + L.wat); h.ba_out = (float *)(ws + L.ba); h.wbt = (float *)(ws + L.wbt); h.bb_out = (float *)(ws + L.bb);
    h.hidden = shape->hidden; h.kv1 = shape->horizon * (shape->num_agents + 1);
    hipLaunchKernelGGL(predictor_split_kernel, dim3(grid), dim3(256), 0, s, wts->wt, (__bf16 *)(ws + L.wp), shape->d, shape->d_x, h);
    e = hipGetLastError();
    if (e != hipSuccess) return pbkv::set_error(PBKV_ERR_DEVICE, "predictor split launch: %s", hipGetErrorString(e));
    return PBKV_OK;
}

int pbkv_predictor_forward(const pbkv_predictor_shape *shape, void *workspace, int64_t workspace_bytes,
                           int32_t max_batch, const void *x, const int32_t *cur_agent, const int32_t *prefix,
                           const int32_t *prefix_len, int32_t batch, float *probs, void *stream) {
    pbkv::clear_error();
    if (int rc = check_shape(shape)) return rc;
    if (max_batch < 1) return pbkv::set_error(PBKV_ERR_RANGE, "max_batch %d is not positive", max_batch);
    if (batch < 0 || batch > max_batch) return pbkv::set_error(PBKV_ERR_RANGE, "batch %d not in [0, max_batch = %d]", batch, max_batch);
    const Layout L = layout(shape, max_batch);
    if (workspace_bytes < L.total)
        return pbkv::set_error(PBKV_ERR_RANGE, "workspace of %lld bytes, %lld needed", (long long)workspace_bytes, (long long)L.total);
    if (int rc = check_dev(workspace, "workspace", 256)) return rc;
    if (batch == 0) return PBKV_OK;
    if (int rc = check_dev(x, "x", 16)) return rc;
    if (int rc = check_dev(cur_agent, "cur_agent", 4)) return rc;
    if (int rc = check_dev(prefix_len, "prefix_len", 4)) return rc;
    if (shape->max_prefix > 0)
        if (int rc = check_dev(prefix, "prefix", 4)) return rc;
    if (int rc = check_dev(probs, "probs", 4)) return rc;

    char *ws = (char *)workspace;
    hipStream_t s = (hipStream_t)stream;
    // cut d_x into slices: about one work-group per CU (never more: a CU holds one), a slice being
    // whole rounds of the waves' groups of k-steps
    const int nw = shape->d == 128 ? 4 : 8, ch = shape->d == 128 ? 3 : 5;
    const int ksteps = shape->d_x / 16, rbs = (batch + 31) / 32;
    int ks = (TARGET_WGS + rbs - 1) / rbs;
    ks = ks > KS_MAX ? KS_MAX : ks;
    const int round_steps = ch * nw;
    const int sps = ((ksteps + ks - 1) / ks + round_steps - 1) / round_steps * round_steps;
    ks = (ksteps + sps - 1) / sps;

    ProjectParams pp;
    pp.x = (const __bf16 *)x; pp.wp = (const __bf16 *)(ws + L.wp);
    pp.partial = (float *)(ws + L.partial);
    pp.batch = batch; pp.bpad = L.bpad; pp.d_x = shape->d_x; pp.steps_per_slice = sps; pp.ksteps = ksteps;
    const dim3 grid(rbs, ks);
    switch (shape->d) {
        case 32: hipLaunchKernelGGL((predictor_project_kernel<1, 8>), grid, dim3(512), 0, s, pp); break;
        case 64: hipLaunchKernelGGL((predictor_project_kernel<2, 8>), grid, dim3(512), 0, s, pp); break;
        default: hipLaunchKernelGGL((predictor_project_kernel<4, 4>), grid, dim3(256), 0, s, pp); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return pbkv::set_error(PBKV_ERR_DEVICE, "predictor projection launch: %s", hipGetErrorString(e));

    HeadParams hp;
    hp.partial = pp.partial; hp.h2 = (const float *)(ws + L.h2); hp.s = (const float *)(ws + L.s);
    hp.wat = (const float *)(ws + L.wat); hp.ba = (const float *)(ws + L.ba);
    hp.wbt = (const float *)(ws + L.wbt); hp.bb = (const float *)(ws + L.bb);
    hp.cur_agent = cur_agent; hp.prefix = prefix; hp.prefix_len = prefix_len; hp.probs = probs;
    hp.batch = batch; hp.slice_floats = (int64_t)L.bpad * shape->d; hp.n_slices = ks; hp.V = shape->num_agents; hp.d = shape->d;
    hp.hidden = shape->hidden; hp.K = shape->horizon; hp.L = shape->max_prefix;
    const int rpb = batch <= HEAD_SMALL_BATCH ? 4 : 8;
    void (*head)(HeadParams) = rpb == 4 ? predictor_head_kernel<4> : predictor_head_kernel<8>;
    hp.kv1 = hp.K * (hp.V + 1);
    hp.inv_K = 65536 / hp.K + 1;
    hp.y1 = head_layer(3 * hp.d, hp.hidden);
    hp.y2 = head_layer(hp.hidden, hp.kv1);
    hp.o = head_lds(rpb, hp.V, hp.d, hp.hidden, hp.kv1, hp.y1, hp.y2);
    const size_t lds_bytes = (size_t)hp.o.total * 4;
    if (lds_bytes > 64 * 1024) {      // above the default limit the kernel has to be told (gfx950 has 160 KiB per work-group)
        hipError_t ea = hipFuncSetAttribute((const void *)head, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (ea != hipSuccess) return pbkv::set_error(PBKV_ERR_DEVICE, "predictor head LDS size %zu: %s", lds_bytes, hipGetErrorString(ea));
    }
    hipLaunchKernelGGL(head, dim3((batch + rpb - 1) / rpb), dim3(HNT), lds_bytes, s, hp);
    e = hipGetLastError();
    if (e != hipSuccess) return pbkv::set_error(PBKV_ERR_DEVICE, "predictor head launch: %s", hipGetErrorString(e));
    return PBKV_OK;
}

}  // extern "C"
