// Block mean-pooling of Q, K, V (Sec. 3.2 "Compression Branch": non-overlapping average
// pooling, here over runs of B consecutive tokens) fused with the re-layout of K and V into
// per-(head, block) MFMA operand tiles for the selection kernel.  One pass over Q, K, V: the
// kernel is HBM-bandwidth bound (reads 3 * n_tok * heads * 64 elements once).
#include "s3r_device.h"
#include "s3r_kernels.h"

namespace s3r {

template <int B> constexpr int kPoolHeads = B < 32 ? 32 / B : 1;

// Eight channels of a row as they are loaded, 16 bytes at a time.
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
    bf16x8 x;
    __device__ __forceinline__ void load(const bf16_t *p) { x = *reinterpret_cast<const bf16x8 *>(p); }
    // the values and their hi parts; zeros for a row that does not exist
    __device__ __forceinline__ void get(bool valid, float (&f)[8], bf16x8 &hi) const
    {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        hi = __builtin_bit_cast(bf16x8, valid ? __builtin_bit_cast(u32x4, x) : u32x4{0u, 0u, 0u, 0u});
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = static_cast<float>(hi[i]);
    }
};
template <> struct Raw8<float> {
    floatx4 a, b;
    __device__ __forceinline__ void load(const float *p)
    {
        a = *reinterpret_cast<const floatx4 *>(p);
        b = *reinterpret_cast<const floatx4 *>(p + 4);
    }
    __device__ __forceinline__ void get(bool valid, float (&f)[8], bf16x8 &hi) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { f[i] = valid ? a[i] : 0.f; f[4 + i] = valid ? b[i] : 0.f; }
#pragma unroll
        for (int i = 0; i < 8; ++i) hi[i] = static_cast<bf16_t>(f[i]);
    }
};

// Operand parts of fp32 inputs: x = hi + lo + O(2^-17 |x|) with hi = bf16(x), lo = bf16(x - hi); with the third part
// lo2 = bf16(x - hi - lo) the sum is x itself (each residual has 8 significant bits fewer than the one before).
// V goes to the matrix pipe as a pair (its products with probabilities in [0, 1] need no more), K as a triple:
// the error of a logit enters the result through an exponential, in absolute terms, so the scores must keep
// all 24 bits of K and Q however large their entries, or those beside them, are.
__device__ __forceinline__ bf16x8 lo_parts(const float (&f)[8], const bf16x8 &hi)
{
    bf16x8 lo;
#pragma unroll
    for (int i = 0; i < 8; ++i) lo[i] = static_cast<bf16_t>(f[i] - static_cast<float>(hi[i]));
    return lo;
}
__device__ __forceinline__ bf16x8 lo2_parts(const float (&f)[8], const bf16x8 &hi, const bf16x8 &lo)
{
    bf16x8 lo2;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        lo2[i] = static_cast<bf16_t>((f[i] - static_cast<float>(hi[i])) - static_cast<float>(lo[i]));
    return lo2;
}

// A 16-byte piece of a tile; PAST: past the L2, where the tiles are more than the caches keep for the kernels that read them (us a
// call, one row at a time, through it / past it: 36 views 453.4 / 453.4, in blocks of 32 411 / 407; 100 views 1215 / 1209, in blocks of 32
// 1163 / 1157; 1000 views, this kernel, 2765 / 2655).  Short sequences are read from there: 8 views, this kernel 23.0 / 21.5, but the one that
// reads the tiles takes as much longer (in blocks of 32 the call 91.4 / 94.5; 16 views 179 / 188).
template <bool PAST> __device__ __forceinline__ void store_tile(bf16_t *dst, const bf16x8 &x)
{
    if constexpr (PAST) __builtin_nontemporal_store(x, reinterpret_cast<bf16x8 *>(dst));
    else *reinterpret_cast<bf16x8 *>(dst) = x;
}

// Whether every thread requests all of its rows at once (and stores the tiles through the L2).  With one load at a time a short
// sequence waits for the memory's latency six times (blocks of 64) where once would do; a long one, whose waves keep the memory
// busy anyway, is faster with the fewer requests on their way, blocks of 128 apart (16 heads, us of this kernel at once / at a time, tiles
// through the L2: 12 views 29.4 / 32.4, 100 views 281 / 270, 1000 views 2924 / 2701; blocks of 128, 300 views 864 / 893; fp32,
// 8 views 43.0 / 45.1, blocks of 128 46.2 / 48.9, 30 views 167.7 / 168.2, 100 views 604 / 606, blocks of 16 563 / 554).  Between them (us a call, at once and through the L2 / at a time and past it; blocks of 64, 32, 4 x 4 windows):
//   12 views, 101 MB   150.4 / 153.9   137.1 / 141.8   233 / 245
//   16 views, 135 MB   194.6 / 196.4   178.6 / 188.0   295 / 309
//   24 views, 203 MB   302.0 / 302.2   289.2 / 282.1   444 / 447
//   30 views, 253 MB   381.2 / 375.7   352.5 / 345.3   556 / 555
//   45 views, 380 MB   559.3 / 553.8   509.6 / 499.1   859 / 857
// From 200 to 270 MB it is one or the other by shape (36 calls of 192 to 256 MiB, at a time / at once: 0.98 to 1.02, in the mean 0.998).
constexpr int64_t kPoolAheadBytes = int64_t(256) << 20;  // of q, k and v

inline bool pool_ahead(int64_t n_tok, int heads, int block, bool is_bf16)
{
    return !is_bf16 || block == 128 || n_tok * heads * (3 * 64 * 2) <= kPoolAheadBytes;
}

// grid: one workgroup per (block j, head h), head fastest; 256 threads.  Blocks of 16 rows: two heads per workgroup,
// which would leave half of its threads without a row otherwise (100 views in 4 x 4 windows: 0.37 -> 0.31 ms, the call
// 3.22 -> 3.17).
// Thread (r0 = tid / 8, c = tid % 8) handles channels 8c..8c+7 of rows r0, r0 + 32, ...
template <typename T, int B, bool REPACK, bool AHEAD>
__global__ __launch_bounds__(256) void pool_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                   const T *__restrict__ v, float *__restrict__ qc,
                                                   float *__restrict__ kc, float *__restrict__ vc,
                                                   bf16_t *__restrict__ kb, bf16_t *__restrict__ vb,
                                                   int64_t n_tok, int heads, int64_t n_blk, TokenMap map,
                                                   InStride in, int64_t lo_off)
{
    // fp32 inputs are re-laid-out as bf16 operand parts: the lo tiles lie lo_off elements after the hi ones, K's
    // third part another lo_off elements on
    constexpr bool PAIRS = REPACK && sizeof(T) == 4;
    constexpr int VS_STRIDE = 72;  // bf16 elements per staged V row (64 + pad: conflict-free columns)
    constexpr int HP = kPoolHeads<B>;     // heads of a workgroup
    constexpr int RT = 32 / HP;           // rows that the threads of a head cover at a time
    __shared__ float red[3][32][65];
    __shared__ bf16_t vs[REPACK ? HP * B : 1][VS_STRIDE];
    __shared__ bf16_t vs_lo[PAIRS ? HP * B : 1][VS_STRIDE];

    const int64_t bid = blockIdx.x;
    const int groups = (heads + HP - 1) / HP;
    const int tid = threadIdx.x;
    const int hh = HP == 1 ? 0 : tid >> 7;
    const int h0 = static_cast<int>(bid % groups) * HP, h = h0 + hh;
    const bool have_head = HP == 1 || h < heads;
    const int64_t j = bid / groups;
    const int c = tid & 7, r0 = (tid >> 3) & (RT - 1);
    const int64_t t0 = j * B;
    const int len = map.block_len(j, B, n_tok);
    const int64_t tile_base = (static_cast<int64_t>(h) * n_blk + j) * (B * 64);

    float acc[3][8];
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[x][i] = 0.f;

    // where chunk c of row r goes: 32-row tiles in operand order; a block of 16 rows is stored as the 16-row half of such a
    // tile, column chunk by column chunk, so that two of them interleave into one tile
    auto k_tile = [&](int r) -> bf16_t * {
        return (B >= 32) ? kb + tile_base + (r >> 5) * kRowTileElems + row_tile_chunk_offset(r & 31, c) : kb + tile_base + (c * 16 + r) * 8;
    };
    // AHEAD: every row of a thread is requested before the first is used; otherwise one load at a time, see pool_ahead.
    // (Ahead: rows and heads that do not exist read one that does.)
    constexpr int NA = AHEAD ? B / RT : 1;
    Raw8<T> rq[NA], rk[NA], rv[NA];
    auto offset_of = [&](int n) -> int64_t {
        const int r = r0 + n * RT;
        return in.at(map.row(r < len ? t0 + r : t0), have_head ? h : h0, heads) + c * 8;
    };
    if constexpr (AHEAD) {
#pragma unroll
        for (int n = 0; n < NA; ++n) {
            const int64_t off = offset_of(n);
            rq[n].load(q + off);
            rk[n].load(k + off);
            rv[n].load(v + off);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int n = 0; n < B / RT; ++n) {
        if (!have_head) break;
        const int r = r0 + n * RT;
        const bool valid = r < len;
        const int64_t off = AHEAD ? 0 : offset_of(n);
        const int na = AHEAD ? n : 0;
        const bool wanted = B > 16 || valid;  // (blocks of 16: slots that windows cut off; 100 views in 4 x 4 windows 330 us, 301 so)
        float f[8];
        bf16x8 hi;
        if (!AHEAD && wanted) rq[na].load(q + off);
        rq[na].get(valid, f, hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[0][i] += f[i];
        if constexpr (!AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            if (wanted) rk[na].load(k + off);
        }
        rk[na].get(valid, f, hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[1][i] += f[i];
        if constexpr (REPACK) {
            bf16_t *dst = k_tile(r);
            store_tile<!AHEAD>(dst, hi);
            if constexpr (PAIRS) {
                const bf16x8 lo = lo_parts(f, hi);
                *reinterpret_cast<bf16x8 *>(dst + lo_off) = lo;
                *reinterpret_cast<bf16x8 *>(dst + 2 * lo_off) = lo2_parts(f, hi, lo);
            }
        }
        if constexpr (!AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            if (wanted) rv[na].load(v + off);
        }
        rv[na].get(valid, f, hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[2][i] += f[i];
        if constexpr (REPACK) {
            *reinterpret_cast<bf16x8 *>(&vs[hh * B + r][c * 8]) = hi;
            if constexpr (PAIRS) *reinterpret_cast<bf16x8 *>(&vs_lo[hh * B + r][c * 8]) = lo_parts(f, hi);
        }
    }
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int i = 0; i < 8; ++i) red[x][hh * RT + r0][c * 8 + i] = acc[x][i];
    __syncthreads();

    if (qc != nullptr) {
        for (int e = tid; e < 192 * HP; e += 256) {
            const int x = (e >> 6) % 3, d = e & 63, hs = e / 192;
            if (HP > 1 && h0 + hs >= heads) break;
            float s = 0.f;
#pragma unroll
            for (int g = 0; g < RT; ++g) s += red[x][hs * RT + g][d];
            float *dst = (x == 0) ? qc : (x == 1) ? kc : vc;
            dst[(static_cast<int64_t>(h0 + hs) * n_blk + j) * 64 + d] = s / static_cast<float>(len);
        }
    }

    if constexpr (REPACK) {
        // V tile, contraction (key) index made contiguous per lane: see tr_tile_key().
        for (int ci = HP == 1 ? tid : tid & 127; ci < B * 8; ci += 256 / HP) {
            if (!have_head) break;
            // (blocks of 16 rows: the two channel tiles of a 16-byte piece one after the other, see small_v_piece)
            const int l = ci & 63, dt = (ci >> 6) & 1, u = ci >> 7;
            const int d = B == 16 ? 32 * dt + (l & 15) : 32 * dt + (l & 31);
            auto row_of = [&](int i) { return hh * B + (B == 16 ? 4 * (l >> 4) + (i & 3) : tr_tile_key(u, l, i)); };
            auto channel_of = [&](int i) { return B == 16 ? d + 16 * (i >> 2) : d; };
            bf16x8 o;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = vs[row_of(i)][channel_of(i)];
            store_tile<!AHEAD>(vb + tile_base + static_cast<int64_t>(ci) * 8, o);
            if constexpr (PAIRS) {
#pragma unroll
                for (int i = 0; i < 8; ++i) o[i] = vs_lo[row_of(i)][channel_of(i)];
                *reinterpret_cast<bf16x8 *>(vb + lo_off + tile_base + static_cast<int64_t>(ci) * 8) = o;
            }
        }
    }
}

template <typename T, int B, bool REPACK, bool AHEAD = true>
static hipError_t run_pool(const void *q, const void *k, const void *v, float *qc, float *kc,
                           float *vc, void *kb, void *vb, int64_t n_tok, int heads, int64_t n_blk,
                           TokenMap map, InStride in, hipStream_t stream)
{
    const int64_t grid = n_blk * ((heads + kPoolHeads<B> - 1) / kPoolHeads<B>);
    const int64_t lo_off = static_cast<int64_t>(heads) * n_blk * B * 64;   // fp32 inputs: [hi tiles | lo tiles | K: lo2 tiles]
    hipLaunchKernelGGL((pool_kernel<T, B, REPACK, AHEAD>), dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                       stream, static_cast<const T *>(q), static_cast<const T *>(k),
                       static_cast<const T *>(v), qc, kc, vc, static_cast<bf16_t *>(kb),
                       static_cast<bf16_t *>(vb), n_tok, heads, n_blk, map, in, lo_off);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void block_lens_kernel(TokenMap map, int block, int64_t n_tok, int64_t n_blk,
                                                         int32_t *__restrict__ blk_len)
{
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (j < n_blk) blk_len[j] = map.block_len(j, block, n_tok);
}

hipError_t launch_block_lens(TokenMap map, int block, int64_t n_tok, int64_t n_blk, int32_t *blk_len,
                             hipStream_t stream)
{
    const int64_t grid = (n_blk + 255) / 256;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(block_lens_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0, stream, map, block, n_tok,
                       n_blk, blk_len);
    return hipGetLastError();
}

hipError_t launch_pool(const void *q, const void *k, const void *v, float *qc, float *kc, float *vc,
                       void *kb, void *vb, int64_t n_tok, int heads, int block, bool is_bf16,
                       TokenMap map, InStride in, hipStream_t stream)
{
    const int64_t n_blk = (n_tok + block - 1) / block;
    if (n_blk * heads > 0x7fffffffLL) return hipErrorInvalidValue;
    if (map.period != 0 && n_tok > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool repack = kb != nullptr;
#define S3R_POOL_CASE(TT, BB, ...) \
    return run_pool<TT, BB, __VA_ARGS__>(q, k, v, qc, kc, vc, kb, vb, n_tok, heads, n_blk, map, in, stream)
    if (!pool_ahead(n_tok, heads, block, is_bf16)) {
        switch (block) {
        case 16: if (repack) S3R_POOL_CASE(bf16_t, 16, true, false); else S3R_POOL_CASE(bf16_t, 16, false, false);
        case 32: if (repack) S3R_POOL_CASE(bf16_t, 32, true, false); else S3R_POOL_CASE(bf16_t, 32, false, false);
        case 64: if (repack) S3R_POOL_CASE(bf16_t, 64, true, false); else S3R_POOL_CASE(bf16_t, 64, false, false);
        }
        return hipErrorInvalidValue;
    }
    if (is_bf16) {
        switch (block) {
        case 16: if (repack) S3R_POOL_CASE(bf16_t, 16, true); else S3R_POOL_CASE(bf16_t, 16, false);
        case 32: if (repack) S3R_POOL_CASE(bf16_t, 32, true); else S3R_POOL_CASE(bf16_t, 32, false);
        case 64: if (repack) S3R_POOL_CASE(bf16_t, 64, true); else S3R_POOL_CASE(bf16_t, 64, false);
        case 128: if (repack) S3R_POOL_CASE(bf16_t, 128, true); else S3R_POOL_CASE(bf16_t, 128, false);
        }
    } else {
        switch (block) {
        case 16: if (repack) S3R_POOL_CASE(float, 16, true); else S3R_POOL_CASE(float, 16, false);
        case 32: if (repack) S3R_POOL_CASE(float, 32, true); else S3R_POOL_CASE(float, 32, false);
        case 64: if (repack) S3R_POOL_CASE(float, 64, true); else S3R_POOL_CASE(float, 64, false);
        case 128: if (repack) S3R_POOL_CASE(float, 128, true); else S3R_POOL_CASE(float, 128, false);
        }
    }
#undef S3R_POOL_CASE
    return hipErrorInvalidValue;
}

}  // namespace s3r
