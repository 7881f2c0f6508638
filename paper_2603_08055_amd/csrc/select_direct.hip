// Selection attention + merge (Sec. 3.2 eq. 6, supplementary Alg. 2; eqs. 5, 7, 8) for blocks of 16 and 32 tokens
// on bf16 MFMA for gfx950: one wave per (query block, head), K/V operands straight from memory to registers.
//
// Work layout.  A query block of 16 (32) tokens fills exactly the 16 (32) columns of one MFMA tile, so a wave owns
// one query block and shares its K/V with nobody: staging units in LDS, as the kernels for larger blocks do to
// share them between waves, would only take the LDS that limits how many waves a CU holds.  The operand-order
// copies written by the pooling kernel are read with plain vector loads, one contiguous run per operand, and the
// waves of a CU hide each other's latency: by their registers 12 for blocks of 16 in bf16, 8 for 32 in bf16 and for 16
// in fp32, 4 for 32 in fp32, against 5 with a 32 KiB ring each (two in fp32).
//   scores      S^T[key][query] = K Q^T: 16x16x32 MFMAs for blocks of 16 (two per block), 32x32x16 for 32 (four)
//   softmax     keys of ONE query per lane: in-lane reductions and one (32) or two (16) exchanges between lanes
//   P.V         O^T[channel][query] += V^T P^T: the probabilities sit in the operand order of 16x16x16 (32x32x16)
// A 16-token block's K tile (pool.hip) is a half tile of the 32-row layout, its V tile has a layout of its own
// (small_v_piece): what the operands need of them is one contiguous KiB per load instruction.  (With the transposed
// tile of 32 rows V took two runs of 256 bytes per load, twice the load instructions: 100 views in 4 x 4 windows 3.06 -> 2.97 ms
// a call, 60 views of clustered keys 1.20 -> 1.14, fp32 30 views in windows 1.48 -> 1.39, 8 views 166 -> 151 us; 60 views of
// i.i.d. keys, where the fabric binds, 1.70 -> 1.72.)
//
// Bound.  The ring kernel ran at 7000 cycles per 64-key unit and wave with one wave per SIMD: a serial chain, the
// matrix pipe 7 % and the vector ALU 30 % busy, half of both for columns that hold no query (blocks of 16).  Now i.i.d.
// keys are delivered at the 7.8 TB/s the fabric has for L2 misses; with keys that neighbouring query blocks share
// (74 % L2 hits at 100 views in 4 x 4 windows) 21 GB of tiles arrive in 1.17 ms, 18 TB/s, with 2.8 waves per SIMD, the
// matrix pipe under 20 % and the vector ALU half busy: what is left is the latency and issue of the loads (a fourth wave per
// SIMD, and no exchange of maxima per unit, measured 0.5 % slower).
//
// Pipelining.  NBU blocks are worked on at a time; the K of the next ones is requested as soon as the scores have
// consumed the registers of the current ones, V after P.V likewise, and the compiler's own counts wait for them.
//
// F32: fp32 q, gate, out and o_sel, K in three and V in two bf16 parts; products as in select_mfma.hip.
#include "s3r_attn_device.h"
#include "s3r_kernels.h"

#include <type_traits>

namespace s3r {

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float max_with_other_rows(float x)  // lanes 16 apart, within each half wave
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float sum_with_other_rows(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int B, bool F32, int NBU, int OCC>
__global__ __launch_bounds__(256, OCC) void select_direct_kernel(
    const void *__restrict__ q_, const bf16_t *__restrict__ kb, const bf16_t *__restrict__ vb,
    const int32_t *__restrict__ idx, const float *__restrict__ o_comp, const void *__restrict__ gate_,
    void *__restrict__ out_, void *__restrict__ o_sel_, float *__restrict__ lse, int64_t n_tok, int64_t n_blk,
    int heads, int kk, float scale_log2, int64_t n_groups, TokenMap qmap, int64_t n_keys, int64_t lse_stride,
    const int32_t *__restrict__ blk_len, const float *__restrict__ o_comp_tok, InStride in, int64_t lo_off, bool whole_heads)
{
    static_assert(B == 16 || B == 32, "one MFMA tile per query block");
    constexpr int NR = B * B / 64;          // score registers of a key block: 4 or 16
    constexpr int KS = B == 16 ? 2 : 4;     // channel steps of the scores: 32 or 16 channels each
    constexpr int NT = B == 16 ? 4 : 2;     // channel tiles of O: 16 or 32 channels each
    constexpr int NKP = F32 ? 3 : 1, NVP = F32 ? 2 : 1;  // operand parts of K (and Q), of V (and P)
    typedef float acc_t __attribute__((ext_vector_type(NR)));

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & (B - 1), g = lane / B;  // the lane's query; which of the lanes that share it
    int h;
    int64_t set;
    int64_t group;  // four query blocks of a head per workgroup
    if (!xcd_item(blockIdx.x, n_groups, heads, whole_heads, h, group)) return;
    set = group * 4 + wave;
    if (set >= n_blk) return;  // (no barriers in this kernel)
    const int64_t t = set * B + col;
    const bool row_valid = blk_len != nullptr ? col < blk_len[set] : t < n_tok;
    const int64_t trow = qmap.row(row_valid ? t : set * B);  // the caller's row of this query

    // Q operands (rows that do not exist repeat the block's first row and are not written)
    bf16x8 qf[NKP][KS];
    {
        const int64_t qo = in.at(trow, h, heads) + 8 * g;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (F32) {
                const float *p = static_cast<const float *>(q_) + qo + (64 / KS) * s;
                const floatx4 a = *reinterpret_cast<const floatx4 *>(p), b = *reinterpret_cast<const floatx4 *>(p + 4);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float f = i < 4 ? a[i & 3] : b[i & 3];
                    qf[0][s][i] = static_cast<bf16_t>(f);
                    const float r1 = f - static_cast<float>(qf[0][s][i]);
                    qf[1][s][i] = static_cast<bf16_t>(r1);
                    qf[2][s][i] = static_cast<bf16_t>(r1 - static_cast<float>(qf[1][s][i]));
                }
            } else {
                qf[0][s] = *reinterpret_cast<const bf16x8 *>(static_cast<const bf16_t *>(q_) + qo + (64 / KS) * s);
            }
        }
    }
    const int32_t *sel = idx + (static_cast<int64_t>(h) * n_blk + set) * kk;
    const bf16_t *kb_h = kb + static_cast<int64_t>(h) * n_blk * (B * 64);
    const bf16_t *vb_h = vb + static_cast<int64_t>(h) * n_blk * (B * 64);
    const unsigned koff = lane * 8;
    const unsigned voff = B == 16 ? small_v_piece(0, g, col) : lane * 8;

    acc_t oacc[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int r = 0; r < NR; ++r) oacc[c][r] = 0.f;
    float m_run = -1e30f, l_run = 0.f;
    const bf16x2 ones = {static_cast<bf16_t>(1.f), static_cast<bf16_t>(1.f)};

    bf16x8 kf[NBU][NKP][KS];
    short4_t vf16[B == 16 ? NBU : 1][NVP][4];
    bf16x8 vf32[B == 32 ? NBU : 1][NVP][4];
    int sel_l, len_l;  // entry and block length of index position base + lane
    auto load_k = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NBU; ++b) {
            const int j = __builtin_amdgcn_readlane(sel_l, u * NBU + b);
#pragma unroll
            for (int p = 0; p < NKP; ++p) {
                const bf16_t *base = kb_h + p * lo_off + static_cast<int64_t>(j) * (B * 64);
#pragma unroll
                for (int s = 0; s < KS; ++s) kf[b][p][s] = *reinterpret_cast<const bf16x8 *>(base + koff + s * 512);
            }
        }
    };
    auto load_v = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NBU; ++b) {
            const int j = __builtin_amdgcn_readlane(sel_l, u * NBU + b);
#pragma unroll
            for (int p = 0; p < NVP; ++p) {
                const bf16_t *base = vb_h + p * lo_off + static_cast<int64_t>(j) * (B * 64);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if constexpr (B == 16) {
                        if ((c & 1) != 0) continue;
                        const short8_t two = *reinterpret_cast<const short8_t *>(base + voff + small_v_piece(c >> 1, 0, 0));
                        vf16[b][p][c] = __builtin_shufflevector(two, two, 0, 1, 2, 3);
                        vf16[b][p][c + 1] = __builtin_shufflevector(two, two, 4, 5, 6, 7);
                    } else vf32[b][p][c] = *reinterpret_cast<const bf16x8 *>(base + voff + c * 512);
                }
            }
        }
    };

    for (int base = 0; base < kk; base += 64) {
        // 64 entries of the index row: lane L holds entry base + L (the last one again past the end, with length 0)
        const int left = kk - base;
        {
            const int e = lane < left ? lane : left - 1;
            int j = sel[base + e];
            j = j < 0 ? 0 : (j >= static_cast<int>(n_blk) ? static_cast<int>(n_blk) - 1 : j);  // a caller's list is not trusted
            sel_l = j;
            const int64_t run = n_keys - static_cast<int64_t>(j) * B;
            len_l = blk_len != nullptr ? blk_len[j] : static_cast<int>(run < B ? run : B);
            if (lane >= left) len_l = 0;
        }
        const unsigned long long is_short = __ballot(len_l < B);
        const int n_units = ((left < 64 ? left : 64) + NBU - 1) / NBU;
        load_k(0);
        load_v(0);
        for (int u = 0; u < n_units; ++u) {
            acc_t sacc[NBU];
#pragma unroll
            for (int b = 0; b < NBU; ++b)
#pragma unroll
                for (int r = 0; r < NR; ++r) sacc[b][r] = 0.f;
            auto mfma_s = [&](int b, const bf16x8 &a, const bf16x8 &x) __attribute__((always_inline)) {
                if constexpr (B == 16) sacc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x, sacc[b], 0, 0, 0);
                else sacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, x, sacc[b], 0, 0, 0);
            };
            // Products of the smaller parts first: what their sums lose is rounding of their own size, and only the products
            // of the high parts are added up at the size of the score.  With each step's products together, o_sel
            // of blocks of 16 was 3.68e-6 off 64 bits on outlier keys (12 x 1374, top-40), 3.57e-6 with q 16 times as large;
            // in this order it is 3.62e-6 and 2.74e-6, in the same time (32x32x16 products, step by step: 3.66e-6, 3.39e-6).
            if constexpr (F32) {
#pragma unroll
                for (int o = 2; o > 0; --o)
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int a = 0; a <= o; ++a)
#pragma unroll
                            for (int b = 0; b < NBU; ++b) mfma_s(b, kf[b][a][s], qf[o - a][s]);
            }
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int b = 0; b < NBU; ++b) mfma_s(b, kf[b][0][s], qf[0][s]);
            if (u + 1 < n_units) load_k(u + 1);
            if (((is_short >> (u * NBU)) & ((1ull << NBU) - 1ull)) != 0ull) {  // keys that do not exist
                asm volatile("" ::: "memory");  // keep this rare path a real branch
#pragma unroll
                for (int b = 0; b < NBU; ++b) {
                    const int len = __builtin_amdgcn_readlane(len_l, u * NBU + b);
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (8 * (r >> 2) + 4 * g + (r & 3) >= len) sacc[b][r] = -INFINITY;
                }
            }
            float mx = sacc[0][0];
#pragma unroll
            for (int b = 0; b < NBU; ++b)
#pragma unroll
                for (int r = 0; r < NR; ++r) mx = fmaxf(mx, sacc[b][r]);
            if constexpr (B == 16) mx = max_with_other_rows(mx);
            const float m_tile = max_with_other_half(mx) * scale_log2;
            const bool grow = m_tile > m_run + kRescaleSlack;
            if (__any(grow)) {  // rare after the first unit: raise the maximum, rescale the accumulators
                const float m_new = grow ? m_tile : m_run;
                const float alpha = fast_exp2(m_run - m_new);
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int r = 0; r < NR; ++r) oacc[c][r] *= alpha;
            }
            float lsum[2] = {0.f, 0.f};
            bf16x4 pf[NVP][NBU][NR / 4];  // registers 4 r4 .. + 3 of block b: keys 8 r4 + 4 g .. + 3
#pragma unroll
            for (int b = 0; b < NBU; ++b)
#pragma unroll
                for (int r = 0; r < NR; r += 2) {
                    const float p0 = fast_exp2(sacc[b][r] * scale_log2 - m_run), p1 = fast_exp2(sacc[b][r + 1] * scale_log2 - m_run);
                    const bf16x2 pr = {static_cast<bf16_t>(p0), static_cast<bf16_t>(p1)};
                    pf[0][b][r >> 2][r & 3] = pr[0];
                    pf[0][b][r >> 2][(r & 3) + 1] = pr[1];
                    if constexpr (F32) {
                        lsum[0] += p0;
                        lsum[1] += p1;
                        pf[1][b][r >> 2][r & 3] = static_cast<bf16_t>(p0 - static_cast<float>(pr[0]));
                        pf[1][b][r >> 2][(r & 3) + 1] = static_cast<bf16_t>(p1 - static_cast<float>(pr[1]));
                    } else {
                        lsum[(r >> 1) & 1] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, lsum[(r >> 1) & 1], false);
                    }
                }
            l_run += lsum[0] + lsum[1];
            auto pv = [&](int b, int vp, int pp) __attribute__((always_inline)) {
                if constexpr (B == 16) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        oacc[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf16[b][vp][c], __builtin_bit_cast(short4_t, pf[pp][b][0]), oacc[c], 0, 0, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {  // chunk c: 16-key step c / 2, channel tile c % 2
                        const bf16x8 p = __builtin_shufflevector(pf[pp][b][2 * (c >> 1)], pf[pp][b][2 * (c >> 1) + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                        oacc[c & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf32[b][vp][c], p, oacc[c & 1], 0, 0, 0);
                    }
                }
            };
#pragma unroll
            for (int b = 0; b < NBU; ++b) {
                pv(b, 0, 0);
                if constexpr (F32) {
                    pv(b, 0, 1);
                    pv(b, 1, 0);
                }
            }
            if (u + 1 < n_units) load_v(u + 1);
        }
    }

    typedef typename std::conditional<F32, float, bf16_t>::type io_t;
    const int64_t o = (trow * heads + h) * 64;
    constexpr int kPairs = NT * NR / 8;  // runs of four channels, two by two
    auto channel = [&](int j) -> int { return B == 16 ? 16 * (2 * j + (g & 1)) + 8 * (g >> 1) : 16 * j + 8 * g; };
    MergeRow<io_t, kPairs> merge;
    merge.load(o_comp_tok != nullptr ? o_comp_tok + ((row_valid ? t : set * B) * heads + h) * 64
               : o_comp != nullptr   ? o_comp + (static_cast<int64_t>(h) * n_blk + set) * 64
                                     : nullptr,
               gate_ != nullptr ? static_cast<const io_t *>(gate_) + o : nullptr, channel);
    float l_tot = sum_with_other_half(l_run);
    if constexpr (B == 16) l_tot = sum_with_other_rows(l_tot);
    const float inv = 1.f / l_tot;
    float os[kPairs][8];
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        float a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // B = 16: a run is a tile; 32: four runs of a tile
            a[e] = (B == 16 ? oacc[2 * j][e] : oacc[(2 * j) >> 2][4 * ((2 * j) & 3) + e]) * inv;
            b[e] = (B == 16 ? oacc[2 * j + 1][e] : oacc[(2 * j + 1) >> 2][4 * ((2 * j + 1) & 3) + e]) * inv;
        }
        if constexpr (B == 16) join_runs_16(a, b, os[j]);
        else join_runs_32(a, b, os[j]);
    }
    if (!row_valid) return;
    if (lse != nullptr && g == 0) lse[static_cast<int64_t>(h) * lse_stride + trow] = (m_run + __builtin_log2f(l_tot)) * kLn2;
    merge.store(os, static_cast<io_t *>(out_) + o, o_sel_ != nullptr ? static_cast<io_t *>(o_sel_) + o : nullptr, channel);
}

template <int B, bool F32, int NBU, int OCC>
static hipError_t run_direct(const SelectArgs &a, hipStream_t stream)
{
    const int64_t groups = (a.n_blk + 3) / 4;
    const bool whole_heads = xcd_whole_heads(a);
    const int64_t grid = xcd_grid(groups, a.heads, whole_heads);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((select_direct_kernel<B, F32, NBU, OCC>), dim3(static_cast<unsigned>(grid)), dim3(256), 0, stream,
                       a.q, static_cast<const bf16_t *>(a.kb), static_cast<const bf16_t *>(a.vb), a.idx, a.o_comp,
                       a.gate, a.out, a.o_sel, a.lse, a.n_tok, a.n_blk, a.heads, a.kk, a.scale * kLog2e, groups, a.qmap,
                       a.n_keys, a.lse_stride, a.blk_len, a.x.o_comp_tok, a.x.in, a.lo_off, whole_heads);
    return hipGetLastError();
}

hipError_t launch_select_direct(const SelectArgs &a, hipStream_t stream)
{
    if (a.kb == nullptr || a.vb == nullptr || a.idx == nullptr || a.kk < 1) return hipErrorInvalidValue;
    if (a.n_keys != a.n_tok || a.n_keys2 != 0 || (!a.is_bf16 && a.lo_off <= 0)) return hipErrorInvalidValue;
    if (a.qmap.period != 0 && a.n_tok > 0x7fffffffLL) return hipErrorInvalidValue;
    // Blocks at a time and waves per SIMD, measured on MI355X (16 heads, top-32; ms of this kernel; in front the
    // kernel with an LDS ring that it took the place of):
    //   blocks of 16, bf16, 100 views in 4 x 4 windows  4.01 | (4, 4) 1.39 (spills)  (4, 3) 1.34  (2, 5) 1.35  (8, 2) 1.40
    //   blocks of 16, bf16, 300 views, i.i.d. keys      8.71 | (4, 3) 6.92: 54 GB of tiles at 7.8 TB/s, all L2 misses
    //   blocks of 32, bf16, 100 views                   2.31 | (2, 3) 1.54 (spills)  (2, 2) 1.24  (1, 4) 1.56  (4, 1) 1.43
    //   blocks of 16, fp32, 60 views                    6.08 | (1, 4) 1.99  (2, 3) 1.80  (4, 2) 1.66  (4, 1) 1.82
    //   blocks of 32, fp32, 60 views                    5.20 | (1, 2) 2.48  (2, 1) 2.15
    // Twice the blocks at a time halve the exchanges and the bookkeeping per score; more than the registers hold
    // spill.  With fewer waves also fewer query blocks are in work per XCD, and more of their units hit its L2.
    if (a.block == 16) return a.is_bf16 ? run_direct<16, false, 4, 3>(a, stream) : run_direct<16, true, 4, 2>(a, stream);
    if (a.block == 32) return a.is_bf16 ? run_direct<32, false, 2, 2>(a, stream) : run_direct<32, true, 2, 1>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace s3r
