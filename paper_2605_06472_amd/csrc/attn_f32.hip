// fp32 prefix-reuse prefill attention on the 32x32x2 fp32 MFMA: for fp32 inputs, where the result must
// agree with the fp64 definition to 1e-5, so there is no reduced-precision contraction anywhere on
// this path.
//
// Work decomposition
//   A row is (suffix token, query head of the KV head's group), numbered token-major, so any head ratio
//   fills the MFMA columns and one new token of a group of G heads already fills G of them.  Work-group =
//   4 waves = (request, KV head, block of 128 rows, range of 32-key tiles); wave w takes 32 of the rows, all
//   four share the K/V tile in LDS.  Ranges shorter than the whole context leave a partial result that
//   attn_f32_merge_kernel folds (see choose_cut_f32 on the host side for when that is done).
//
// Orientation as in the bf16 kernel: S^T = K Q^T, O^T = V^T P^T.  The contraction indices are labels, so
//   * K is read 16 bytes at a time: lane (li, lh) holds K[li][8q + 4 lh .. +3], which feeds four MFMAs whose
//     k pair is (d, d + 4); Q is held in the same order;
//   * register r of the scores is key 8(r/4) + r%4 in lanes lh = 0 and that + 4 in lanes lh = 1: exactly
//     the B operand of one PV step, no exchange between lanes;
//   * V is read D/32 floats at a time: lane li holds d = li D/32 .. of its key, one per O block, so that
//     block b's MFMA row m is d = m D/32 + b and a lane stores D/32 consecutive floats of the result.
// K rows are stored with their 16-byte chunks XORed by the row number (reads of 16 consecutive rows touch
// every bank once); V reads are contiguous per half wave.
//
// What bounds it: an MFMA of this shape occupies the matrix pipe for 64 cycles, a tile step of a wave is
// D of them (3.9 us at D = 128), against D / 4 LDS reads and 16 exponentials; K/V of the next tile are
// fetched into registers meanwhile.  Small calls are bound by the launch and its dependent fetches.
// Before, one query row per lane on the vector ALU, one wave per 64 rows of one head, K/V read back from LDS
// as broadcasts: 256 + 64 tokens, 2/1 heads of 64 took 208 us, now 12.5 per call (two kernels of 9.1 and 3.4 us); four
// requests of 2048 + 256, 8/2 heads of 128 (9.1 GFLOP) run at 86 TFLOP/s, a large fp32 matrix product at 154.
#include "pbkv_internal.h"

namespace pbkv {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int F32_ROWS = 128;  // (token, head) rows per work-group

int attn_f32_block_rows() { return F32_ROWS; }
// floats of one partial result: the O registers of four waves [wave][register][lane][O block], then
// (reference, row sum) per row
int64_t attn_f32_partial_floats(int head_dim) { return (int64_t)F32_ROWS * (head_dim + 2); }

template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_f32_kernel(AttnParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int DB = D / 32;
    constexpr int CPR = D / 4;                     // 16-byte chunks per row
    constexpr int RPP = 256 / CPR;                 // rows the work-group fetches per pass
    constexpr int NP = F32_KEYS / RPP;             // passes (loads of K, and of V, per thread and tile)
    __shared__ __attribute__((aligned(16))) float sK[2][F32_KEYS][D];
    __shared__ __attribute__((aligned(16))) float sV[2][F32_KEYS][D];
    const int tid = threadIdx.x, l = tid & 63, li = l & 31, lh = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = blockIdx.x % p.Hkv;
    const int tile = blockIdx.x / p.Hkv;
    const TileDesc td = p.tiles[tile];
    RangeDesc rd{-1, 0, INT32_MAX, 0};
    if (p.ranges != nullptr) rd = p.ranges[tile];
    if (p.mirror != nullptr && kvh == 0 && tid == 0) {
        p.mirror[tile] = td;
        if (p.ranges != nullptr) p.mirror_ranges[tile] = rd;
    }
    const int G = p.Hq / p.Hkv;
    const int n_rows = td.new_len * G;
    const int wrow0 = td.tok0 + 32 * w;            // tok0: first row of the block
    const bool active = wrow0 < n_rows;            // wave-uniform
    const int row = min(wrow0 + li, n_rows - 1);
    const int tok = row / G, head = kvh * G + row % G;
    const int last_tok = (min(td.tok0 + F32_ROWS, n_rows) - 1) / G;
    const int n_keys = td.prefix_len + last_tok + 1;          // keys visible to the block's last row
    const int my_keys = td.prefix_len + tok + 1;
    const int min_keys = td.prefix_len + min(wrow0, n_rows - 1) / G + 1;   // ... to the wave's first row
    const int kt0 = rd.kt0, kt1 = min(rd.kt1, (n_keys + F32_KEYS - 1) / F32_KEYS);

    const int32_t *bt = p.block_table + (int64_t)td.req * p.max_pages;
    const float *pool = (const float *)p.kv_pool + (int64_t)kvh * 16 * D;
    const float *kn = (const float *)p.k_new + (td.row0 * p.Hkv + kvh) * D;
    const float *vn = (const float *)p.v_new + (td.row0 * p.Hkv + kvh) * D;
    const int lrow = tid / CPR, lc = tid % CPR;
    f32x4 kr[NP], vr[NP];
    auto fetch = [&](int t) {
        int pg[NP];
#pragma unroll
        for (int i = 0; i < NP; i++) {
            const int j = t * F32_KEYS + i * RPP + lrow;
            pg[i] = j < td.prefix_len ? bt[j >> 4] : 0;
        }
#pragma unroll
        for (int i = 0; i < NP; i++) {
            const int j = t * F32_KEYS + i * RPP + lrow;
            kr[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            vr[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (j < td.prefix_len) {
                const int q = pg[i] < 0 ? 0 : (pg[i] >= p.num_pages ? p.num_pages - 1 : pg[i]);
                const float *src = pool + ((int64_t)q * 2 * p.Hkv * 16 + (j & 15)) * D + lc * 4;
                kr[i] = *(const f32x4 *)src;
                vr[i] = *(const f32x4 *)(src + (int64_t)p.Hkv * 16 * D);
            } else if (j < n_keys) {
                const int64_t off = (int64_t)(j - td.prefix_len) * p.Hkv * D + lc * 4;
                kr[i] = *(const f32x4 *)(kn + off);
                vr[i] = *(const f32x4 *)(vn + off);
            }
        }
    };
    auto put = [&](int b) {
#pragma unroll
        for (int i = 0; i < NP; i++) {
            const int r = i * RPP + lrow;
            *(f32x4 *)&sK[b][r][(lc ^ (r & 15)) * 4] = kr[i];
            *(f32x4 *)&sV[b][r][lc * 4] = vr[i];
        }
    };
    fetch(kt0);

    f32x4 q[D / 8];
    {
        const float *qf = (const float *)p.q + ((td.row0 + tok) * p.Hq + head) * D + 4 * lh;
#pragma unroll
        for (int i = 0; i < D / 8; i++) q[i] = *(const f32x4 *)(qf + 8 * i);
    }
    const float c = 1.4426950408889634f * rsqrtf((float)D);
    f32x16 O[DB];
#pragma unroll
    for (int b = 0; b < DB; b++)
#pragma unroll
        for (int r = 0; r < 16; r++) O[b][r] = 0.f;
    // reference in log2 units (from the lowest finite value, not -inf: a range may begin with keys whose scores are
    // -inf, which count nothing against it); this lane's share of the row sum
    float M = -__FLT_MAX__, lsum = 0.f;

    for (int t = kt0; t < kt1; t++) {
        const int b = (t - kt0) & 1;
        put(b);
        __syncthreads();                           // tile t is in buffer b; every wave is done with the tile before the last
        if (t + 1 < kt1) fetch(t + 1);
        if (!active) continue;
        // Four chains (at D = 128 two at a time: four accumulators do not fit): a chain's rounding error grows with its sum, and with
        // two chains short contexts came out 1.1 to 1.3 times as far from fp64 as four chains on the vector ALU (2.06e-7 against
        // 1.60e-7 at four of 16 + 8 tokens; now 1.51e-7).  That costs 1.5 % of a call in the mean of 100 drawn ones, 4 % at
        // most (at D = 64 it was half a percent more with the halves one after the other).
        f32x16 S, S1, S2, S3;
        auto chains = [&](int half, f32x16 &a, f32x16 &b2) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; r++) { a[r] = 0.f; b2[r] = 0.f; }
#pragma unroll
            for (int i = half * D / 16; i < (half + 1) * D / 16; i++) {
                const f32x4 k = *(const f32x4 *)&sK[b][li][((2 * i + lh) ^ (li & 15)) * 4];
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    a = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e], q[i][e], a, 0, 0, 0);
                    b2 = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e + 1], q[i][e + 1], b2, 0, 0, 0);
                }
            }
        };
        chains(0, S2, S3);
        if constexpr (D == 128) {
#pragma unroll
            for (int r = 0; r < 16; r++) S2[r] += S3[r];
        }
        chains(1, S, S1);
#pragma unroll
        for (int r = 0; r < 16; r++) S[r] = D == 128 ? (S[r] + S1[r]) + S2[r] : (S[r] + S1[r]) + (S2[r] + S3[r]);
        if ((t + 1) * F32_KEYS > min_keys) {
            const int rel = my_keys - t * F32_KEYS - 4 * lh;
#pragma unroll
            for (int r = 0; r < 16; r++)
                if (8 * (r >> 2) + (r & 3) >= rel) S[r] = -INFINITY;
        }
        float mx = S[0];
#pragma unroll
        for (int r = 1; r < 16; r++) mx = fmaxf(mx, S[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c;
        if (__any(mx > M)) {
            const float newM = fmaxf(M, mx);
            const float alpha = __builtin_amdgcn_exp2f(M - newM);
            M = newM;
            lsum *= alpha;
#pragma unroll
            for (int x = 0; x < DB; x++)
#pragma unroll
                for (int r = 0; r < 16; r++) O[x][r] *= alpha;
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
            S[r] = __builtin_amdgcn_exp2f(fmaf(S[r], c, -M));
            lsum += S[r];
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const float *v = &sV[b][8 * (r >> 2) + (r & 3) + 4 * lh][li * DB];
            if constexpr (DB == 4) {
                const f32x4 a = *(const f32x4 *)v;
#pragma unroll
                for (int x = 0; x < DB; x++) O[x] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x], S[r], O[x], 0, 0, 0);
            } else {
                const f32x2 a = *(const f32x2 *)v;
#pragma unroll
                for (int x = 0; x < DB; x++) O[x] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x], S[r], O[x], 0, 0, 0);
            }
        }
    }
    if (!active || wrow0 + li >= n_rows) return;
    lsum += __shfl_xor(lsum, 32, 64);
    typedef __attribute__((ext_vector_type(DB))) float f32xd;
    if (rd.part >= 0) {
        float *ps = p.partial + ((int64_t)rd.part * p.Hkv + kvh) * F32_ROWS * (D + 2);
#pragma unroll
        for (int r = 0; r < 16; r++) {
            f32xd v;
#pragma unroll
            for (int x = 0; x < DB; x++) v[x] = O[x][r];
            *(f32xd *)(ps + ((w * 16 + r) * 64 + l) * DB) = v;
        }
        if (lh == 0) *(f32x2 *)(ps + F32_ROWS * D + (w * 32 + li) * 2) = f32x2{M, lsum};
        return;
    }
    const float inv = 1.0f / lsum;
    float *of = (float *)p.out + ((td.row0 + tok) * p.Hq + head) * D;
#pragma unroll
    for (int r = 0; r < 16; r++) {
        f32xd v;
#pragma unroll
        for (int x = 0; x < DB; x++) v[x] = O[x][r] * inv;
        *(f32xd *)(of + (8 * (r >> 2) + 4 * lh + (r & 3)) * DB) = v;
    }
#endif
}

// Folds the partial results of the row blocks whose keys were dealt out to several work-groups.  Work-group =
// (row block, wave of the main kernel, four of its 16 O registers, KV head), wave = register, lane = lane.
template <int D>
__global__ __launch_bounds__(256) void attn_f32_merge_kernel(AttnParams p) {
    constexpr int DB = D / 32;
    typedef __attribute__((ext_vector_type(DB))) float f32xd;
    int bid = blockIdx.x;
    const int kvh = bid % p.Hkv;
    bid /= p.Hkv;
    const int r = 4 * (bid & 3) + (threadIdx.x >> 6), w = (bid >> 2) & 3;
    const int m = bid >> 4;
    const MergeDesc md = p.merges[m];
    if (p.mirror_merges != nullptr && kvh == 0 && (bid & 15) == 0 && threadIdx.x == 0) p.mirror_merges[m] = md;
    const int l = threadIdx.x & 63, li = l & 31, lh = l >> 5;
    const int G = p.Hq / p.Hkv;
    const int row = md.tok0 + 32 * w + li;
    if (row >= md.new_len * G) return;
    const int64_t stride = (int64_t)p.Hkv * F32_ROWS * (D + 2);
    const float *ps = p.partial + ((int64_t)md.part0 * p.Hkv + kvh) * F32_ROWS * (D + 2);
    const float *ml = ps + F32_ROWS * D + (w * 32 + li) * 2;
    const float *po = ps + ((w * 16 + r) * 64 + l) * DB;
    f32xd num;
    float den;
    merge_parts<MERGE_AHEAD>(ml, po, stride, md.n_parts, num, den);
    const float inv = 1.0f / den;
#pragma unroll
    for (int x = 0; x < DB; x++) num[x] *= inv;
    const int tok = row / G, head = kvh * G + row % G;
    *(f32xd *)((float *)p.out + ((md.row0 + tok) * p.Hq + head) * D + (8 * (r >> 2) + 4 * lh + (r & 3)) * DB) = num;
}

template <int D>
static hipError_t launch_f32(const AttnParams &p, hipStream_t s) {
    hipLaunchKernelGGL(attn_f32_kernel<D>, dim3((unsigned)p.n_tiles * p.Hkv), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.n_merges == 0) return e;
    hipLaunchKernelGGL(attn_f32_merge_kernel<D>, dim3((unsigned)p.n_merges * 16 * p.Hkv), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_attn_f32(const AttnParams &p, int head_dim, hipStream_t s) {
    if (p.n_tiles == 0) return hipSuccess;
    return head_dim == 64 ? launch_f32<64>(p, s) : launch_f32<128>(p, s);
}

}  // namespace pbkv
