// Compression branch and TopK (Sec. 3.2, eqs. 3-4 and "Selection Branch") for short sequences of pooled blocks, in one
// launch: block scores, compressed attention and the index lists straight from the pooled means.
//
// What bounds it.  With a few hundred pooled blocks the products are a fraction of a microsecond; what the sweeps of
// compress.hip cost there is a chain of five launches (statistics, operand tiles, threshold sweep, filter sweep,
// candidates), each a few waves long and each waiting for the one before.  Here a row of scores fits in LDS, so no bound,
// no candidates and no operand tiles are needed: one workgroup takes 16 pooled queries of a head and goes through
//   scores    S = Qc Kc^T, 16 keys per wave and step, fp32 MFMAs (16x16x4) on the fp32 means themselves
//   rows      one wave per query: softmax over its row, and the k largest scores by a bitwise search with wave ballots;
//             keys too close to the k-th score to tell are compared by the dot product that topk_candidates_kernel takes,
//             so that the index lists are the same as by the sweeps
//   P.V       Oc' = P Vc, each wave 16 channels of a quarter of the keys, partial sums added up in LDS
// The fp32 matrix pipe is 1/16 as fast as the bf16 one, and still not what the time goes into; scores and
// probabilities are fp32 throughout, at least as exact as the two-part and fp16 scores of the sweeps.
// Two workgroups on a CU cover each other's latency (one from 513 to 1024 blocks, with a row of 1024 scores for all of them
// and the partial sums beside it: 645 blocks, 16 heads 431 us a call, now 409; 724 blocks 487 and 464; 965, 9 heads 403 and
// 385): hence 64 registers, a size of its own up to 768 blocks, and above it the partial sums in the probabilities' place.
// Whole calls, the launches that this one took the place of -> this one (MI355X): 4 x 256 tokens, 2 heads, fp32 51.5 ->
// 21 us; 7 x 777, 5 heads, blocks of 32 59.5 -> 33; 8 x 1374, 16 heads 133 -> 103.  Where the line to the sweeps lies:
// compress_small_takes.
#include "s3r_device.h"
#include "s3r_kernels.h"

namespace s3r {

constexpr int kSmallQ = 16;      // pooled queries of a workgroup
constexpr int kSmallWaves = 16;  // one per query in the row phase

// Maximum and sum over the 64 lanes, the same value in all of them, on the vector ALU: exchanges inside a row of 16 lanes by
// DPP, the rows by lane swaps (a shuffle through LDS takes over 100 cycles, and a row phase has a few dozen in a chain).
template <int CTRL> __device__ __forceinline__ float dpp(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

template <typename F> __device__ __forceinline__ float wave_reduce(float x, F &&f)
{
    x = f(x, dpp<0xB1>(x));   // lanes 1 apart: quad_perm [1, 0, 3, 2]
    x = f(x, dpp<0x4E>(x));   // 2 apart: quad_perm [2, 3, 0, 1]
    x = f(x, dpp<0x141>(x));  // the other quad of 8: row_half_mirror
    x = f(x, dpp<0x140>(x));  // the other 8 of 16: row_mirror
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

__device__ __forceinline__ float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }

// NV: score registers of a lane, n_blk <= 64 NV.  grid: (ceil(n_blk / 16), heads)
template <int NV>
__global__ __launch_bounds__(kSmallWaves * 64, 8) void compress_small_kernel(
    const float *__restrict__ qc, const float *__restrict__ kc, const float *__restrict__ vc,
    float *__restrict__ o_comp, int32_t *__restrict__ idx, int n_blk, int k, float scale_log2,
    const unsigned long long *__restrict__ forced_words)
{
    // (+ 4: the rows that a wave writes or reads at a time start in different banks, 16-byte aligned)
    constexpr int kStride = NV * 64 + 4;
    __shared__ __attribute__((aligned(16))) float s[kSmallQ][kStride];       // scores, then probabilities
    // P.V of a quarter of the keys each; in the place of the probabilities where two workgroups do not fit a CU otherwise
    constexpr bool kInPlace = NV > 12;
    __shared__ float part_room[kInPlace ? 1 : 4][kSmallQ][68];
    auto part = kInPlace ? reinterpret_cast<float (*)[kSmallQ][68]>(&s[0][0]) : part_room;
    static_assert(!kInPlace || sizeof(s) >= 4 * kSmallQ * 68 * sizeof(float), "partial sums in the probabilities' place");
    __shared__ float inv_sum[kSmallQ];
    __shared__ float key_norm2[kSmallWaves];  // largest squared norm of the keys that each wave scored

    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.y, q0 = blockIdx.x * kSmallQ;
    const int64_t head = static_cast<int64_t>(h) * n_blk * 64;
    const int n_tiles = (n_blk + 15) / 16;

    // ---- scores.  Operands of step t: channel 16 g + t of row `col`, so that a lane reads 64 contiguous bytes of a row
    // (the order of the channels in a sum is free).  Rows past the end repeat the last one; nothing of them is kept.
    {
        float a[16];
        const float *qrow = qc + head + static_cast<int64_t>(q0 + col < n_blk ? q0 + col : n_blk - 1) * 64 + 16 * g;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const floatx4 f = *reinterpret_cast<const floatx4 *>(qrow + 4 * c);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[4 * c + i] = f[i];
        }
        float kn2 = 0.f;
        for (int kt = wave; kt < n_tiles; kt += kSmallWaves) {
            const int key = kt * 16 + col;
            const float *krow = kc + head + static_cast<int64_t>(key < n_blk ? key : n_blk - 1) * 64 + 16 * g;
            floatx4 f[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) f[c] = *reinterpret_cast<const floatx4 *>(krow + 4 * c);
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 16; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], f[t >> 2][t & 3], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) s[4 * g + r][key] = acc[r];
            float n2 = 0.f;
#pragma unroll
            for (int t = 0; t < 16; ++t) n2 = fmaf(f[t >> 2][t & 3], f[t >> 2][t & 3], n2);
            n2 += __shfl_xor(n2, 16, 64);
            n2 += __shfl_xor(n2, 32, 64);
            kn2 = fmaxf(kn2, n2);
        }
        kn2 = wave_max(kn2);
        if (lane == 0) key_norm2[wave] = kn2;
    }
    // Values of the first steps of P.V, requested early: their latency runs under the row phase.
    const int ct = wave & 3, kq = wave >> 2;  // 16 channels; every fourth run of 16 keys
    constexpr int kEarly = NV < 4 ? NV : NV < 12 ? 4 : NV < 16 ? 3 : 1;  // (what 64 registers hold)
    float v[kEarly][4];
    const float *vcol = vc + head + 16 * ct + col;
    auto value = [&](int run, int i) -> float {
        const int key = run * 16 + 4 * g + i;
        return key < n_blk ? vcol[static_cast<int64_t>(key) * 64] : 0.f;
    };
#pragma unroll
    for (int e = 0; e < kEarly; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[e][i] = value(kq + 4 * e, i);
    __syncthreads();

    // ---- one row per wave
    const int row = q0 + wave;
    {
        float x[NV];
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const int key = 64 * t + lane;
            x[t] = key < n_blk ? s[wave][key] : -INFINITY;
            mx = fmaxf(mx, x[t]);
        }
        mx = wave_max(mx);
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < NV; ++t) {  // (keys that do not exist: probability 0)
            const float p = fast_exp2((x[t] - mx) * scale_log2);
            s[wave][64 * t + lane] = p;
            sum += p;
        }
        sum = wave_sum(sum);
        if (lane == 0) inv_sum[wave] = 1.f / sum;
        if (k > 0 && row < n_blk) {  // wave-uniform
            // order-preserving keys; 0 for blocks that do not take part: past the end, forced (Sec. 3.3), or with a score
            // that is not a number (which is above no bound in the sweeps either)
            uint32_t key[NV];
#pragma unroll
            for (int t = 0; t < NV; ++t) {
                uint32_t o = order_key(x[t]);
                o = o > 1u ? o : 1u;
                bool out = 64 * t + lane >= n_blk || x[t] != x[t];
                if (forced_words != nullptr && 64 * t < n_blk) out = out || ((forced_words[t] >> lane) & 1ull) != 0ull;
                key[t] = out ? 0u : o;
            }
            // k-th largest key, bit by bit; done as soon as exactly k keys are at or above the trial value
            auto search = [&](uint32_t &T) __attribute__((always_inline)) -> bool {
                T = 0u;
                for (int bit = 31; bit >= 0; --bit) {
                    const uint32_t trial = T | (1u << bit);
                    int c = 0;
#pragma unroll
                    for (int t = 0; t < NV; ++t) c += __popcll(__ballot(key[t] >= trial));
                    if (c >= k) T = trial;
                    if (c == k) return true;
                }
                return false;
            };
            uint32_t T;
            bool exact = search(T);
            // This score and the one of topk_candidates_kernel differ by at most eps = 72 2^-24 |q||k| (64 roundings in a row
            // here, 8 there: chains of 4 and a tree of 16).  Keys more than 2 eps above the k-th score are in by
            // either, those more than 2 eps below are out; if others lie between than just as many as are wanted, the scores of
            // topk_candidates_kernel decide among them.  (Outlier keys widen the band for their head, all but equal ones put every
            // key into it: 500 blocks, 16 heads 296 and 375 us a call, 292 on clustered keys; by the sweeps 330, 512 and 322.)
            {
                const float qv = qc[head + static_cast<int64_t>(row) * 64 + lane];
                const float kn2 = wave_max(key_norm2[lane & (kSmallWaves - 1)]);
                const float two_eps = (1.f / 131072.f) * 1.15f * __builtin_sqrtf(wave_sum(qv * qv)) * __builtin_sqrtf(kn2) + 1e-36f;
                // the k-th score itself: the smallest taken
                uint32_t kth_key = 0xff800000u;  // (of +inf)
#pragma unroll
                for (int t = 0; t < NV; ++t)
                    if (key[t] >= T && key[t] != 0u) kth_key = kth_key < key[t] ? kth_key : key[t];
                const float kth = -wave_max(-key_to_float(kth_key));
                // (bounds as keys: the scores themselves need no registers beside them)
                const uint32_t above = order_key(kth + two_eps), below = order_key(kth - two_eps);
                int n_from = 0;
#pragma unroll
                for (int t = 0; t < NV; ++t) n_from += __popcll(__ballot(key[t] >= below && key[t] != 0u));
                if (n_from > k && two_eps == two_eps) {  // (rare)
                    const int sub = lane & 15;
                    const floatx4 q4 = *reinterpret_cast<const floatx4 *>(qc + head + static_cast<int64_t>(row) * 64 + 4 * sub);
#pragma unroll
                    for (int t = 0; t < NV; ++t) {
                        const bool in = key[t] > above, near = !in && key[t] >= below && key[t] != 0u;
                        key[t] = in ? 0xffffffffu : 0u;
                        unsigned long long m = __ballot(near);
                        while (m != 0ull) {  // four at a time, 16 lanes each, in the order of operations of that kernel
                            int l4[4];
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                l4[i] = m != 0ull ? __ffsll(static_cast<long long>(m)) - 1 : -1;
                                m &= m - 1ull;  // (0 stays 0)
                            }
                            const int mine = g == 0 ? l4[0] : g == 1 ? l4[1] : g == 2 ? l4[2] : l4[3];
                            const floatx4 k4 = *reinterpret_cast<const floatx4 *>(
                                kc + head + static_cast<int64_t>(64 * t + (mine < 0 ? l4[0] : mine)) * 64 + 4 * sub);
                            float dot = 0.f;
#pragma unroll
                            for (int i = 0; i < 4; ++i) dot = __builtin_fmaf(q4[i], k4[i], dot);
                            dot += __shfl_xor(dot, 1, 64);
                            dot += __shfl_xor(dot, 2, 64);
                            dot += __shfl_xor(dot, 4, 64);
                            dot += __shfl_xor(dot, 8, 64);
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const uint32_t o = order_key(__shfl(dot, 16 * i, 64));
                                if (lane == l4[i]) key[t] = o > 1u ? (o < 0xfffffffeu ? o : 0xfffffffeu) : 1u;
                            }
                        }
                    }
                    exact = search(T);
                }
            }
            int ties = n_blk;  // how many keys equal to T are taken, the smallest indices first
            if (!exact) {
                ties = k;
#pragma unroll
                for (int t = 0; t < NV; ++t) ties -= __popcll(__ballot(key[t] > T));
            }
            int n_out = 0, n_eq = 0;
            int32_t *dst = idx + (static_cast<int64_t>(h) * n_blk + row) * k;
#pragma unroll
            for (int t = 0; t < NV; ++t) {
                const bool eq = key[t] == T && T != 0u;  // (T = 0: fewer than k blocks take part)
                const unsigned long long eq_mask = __ballot(eq);
                const bool take = key[t] > T || (eq && n_eq + lanes_below(eq_mask) < ties);
                const unsigned long long mask = __ballot(take);
                if (take) dst[n_out + lanes_below(mask)] = 64 * t + lane;
                n_out += __popcll(mask);
                n_eq += __popcll(eq_mask);
            }
            for (int i = n_out + lane; i < k; i += 64) dst[i] = 0;  // keep the row in range
        }
    }
    __syncthreads();

    // ---- P.V: 16 keys per step, key 4 g + i of the run in MFMA i
    {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        auto step = [&](int run, const float (&w)[4]) __attribute__((always_inline)) {
            const floatx4 p = *reinterpret_cast<const floatx4 *>(&s[col][run * 16 + 4 * g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(p[i], w[i], acc, 0, 0, 0);
        };
#pragma unroll
        for (int e = 0; e < kEarly; ++e)
            if (kq + 4 * e < n_tiles) step(kq + 4 * e, v[e]);  // wave-uniform
        for (int run = kq + 4 * kEarly; run < n_tiles; run += 4) {
            float w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = value(run, i);
            step(run, w);
        }
        if constexpr (kInPlace) __syncthreads();  // every wave has read its probabilities
#pragma unroll
        for (int r = 0; r < 4; ++r) part[kq][4 * g + r][16 * ct + col] = acc[r];
    }
    __syncthreads();
    if (row < n_blk) {
        const float o = (part[0][wave][lane] + part[1][wave][lane]) + (part[2][wave][lane] + part[3][wave][lane]);
        o_comp[head + static_cast<int64_t>(row) * 64 + lane] = o * inv_sum[wave];
    }
}

hipError_t launch_compress_small(const float *qc, const float *kc, const float *vc, float *o_comp, int32_t *idx,
                                 int64_t n_blk, int heads, int k, float scale, const unsigned long long *forced_words,
                                 hipStream_t stream)
{
    if (n_blk < 1 || n_blk > kSmallMaxBlk || heads < 1 || heads > 65535 || k < 0 || k > n_blk) return hipErrorInvalidValue;
    if (k > 0 && idx == nullptr) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>((n_blk + kSmallQ - 1) / kSmallQ), static_cast<unsigned>(heads));
#define S3R_SMALL(NV)                                                                                                   \
    if (n_blk <= (NV) * 64) {                                                                                           \
        hipLaunchKernelGGL(compress_small_kernel<NV>, grid, dim3(kSmallWaves * 64), 0, stream, qc, kc, vc, o_comp, idx, \
                           static_cast<int>(n_blk), k, scale * kLog2e, forced_words);                                   \
        return hipGetLastError();                                                                                       \
    }
    S3R_SMALL(1)
    S3R_SMALL(2)
    S3R_SMALL(4)
    S3R_SMALL(8)
    S3R_SMALL(12)
    S3R_SMALL(16)
#undef S3R_SMALL
    return hipErrorInvalidValue;
}

}  // namespace s3r
