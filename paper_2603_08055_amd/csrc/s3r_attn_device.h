// Device-side helpers of the bf16 MFMA attention kernels (selection and dense): the LDS-direct load,
// explicit vmcnt waits, exchanges between the two halves of a wave, and the constants of the 64-key unit.
#pragma once
#include "s3r_device.h"
#include "s3r_kernels.h"

namespace s3r {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kRescaleSlack = 8.0f;
// A lane's probabilities of a unit add up to more than this if one of them is above 2^kRescaleSlack (rounded to bf16).
constexpr float kMaxUnitSum = 255.0f;
constexpr int kUnitKeys = 64;
constexpr int kUnitElems = kUnitKeys * 64;  // bf16 elements of one K (or V) unit: 8 KiB

__device__ __forceinline__ float max_with_other_half(float x)
{
    // v_permlane32_swap exchanges the two half-waves: one VALU instruction, no LDS traffic
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float sum_with_other_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One LDS-direct load: 64 lanes x 16 bytes from `src` (per-lane address) to LDS byte address
// `lds_byte` (wave-uniform) + 16 * lane.  Counted by vmcnt like any vector memory load.
__device__ __forceinline__ void lds_dma_16(const void *src, unsigned lds_byte)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_byte)
                 : "memory", "m0");
}

// The same with a wave-uniform start address and a byte offset per lane: no address arithmetic in vector registers.
__device__ __forceinline__ void lds_dma_16_x1(const void *base, unsigned voff, unsigned lds_byte)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds_byte)
                 : "memory", "m0");
}

// Two consecutive 1 KiB chunks, see lds_dma_16_x4.
__device__ __forceinline__ void lds_dma_16_x2(const void *base, unsigned voff, unsigned lds_byte)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %1\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:1024"
                 ::"v"(voff), "s"(base), "s"(lds_byte)
                 : "memory", "m0");
}

// Four consecutive 1 KiB chunks of a contiguous run with a wave-uniform start address: lane L's 16 bytes of chunk
// c come from base + voff + c KiB (voff = 16 L, or 16 L + 4096 for the second half of an 8 KiB run: the
// constant offset of the instruction reaches 4095 bytes) and land at LDS byte lds_byte + c KiB + 16 L: the
// instruction's constant offset moves the LDS address along with the global one, so M0 is set once.
__device__ __forceinline__ void lds_dma_16_x4(const void *base, unsigned voff, unsigned lds_byte)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %1\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:2048\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:3072"
                 ::"v"(voff), "s"(base), "s"(lds_byte)
                 : "memory", "m0");
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// ---- merge with the compressed branch and store (eqs. 5, 7, 8) ---------------------------------
// The end of a selection kernel: out = g o_comp + (1 - g) o_sel for the lane's channels of its row, and o_sel itself
// where it is wanted.  An MFMA leaves a lane runs of four channels; two lanes of a query exchange halves of two runs (join) and then
// hold eight channels in a row each, in pairs of runs j = 0 .. NP - 1: 16 bytes per load and store in bf16, half as many of them.
// All loads are issued before the first value is used (load), where one run after the other waited out a memory latency, and the
// stores before it, eight times over (2.2 of 10 us of the fp32 kernel on 4 views of 256 rows).
template <typename IO> struct Io8;
template <> struct Io8<bf16_t> {
    bf16x8 x;
    __device__ __forceinline__ void load(const bf16_t *p) { x = *reinterpret_cast<const bf16x8 *>(p); }
    __device__ __forceinline__ float get(int i) const { return static_cast<float>(x[i]); }
    static __device__ __forceinline__ void store(bf16_t *p, const float (&f)[8])
    {
        bf16x8 r;
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = static_cast<bf16_t>(f[i]);
        *reinterpret_cast<bf16x8 *>(p) = r;
    }
};
template <> struct Io8<float> {
    floatx4 a, b;
    __device__ __forceinline__ void load(const float *p)
    {
        a = *reinterpret_cast<const floatx4 *>(p);
        b = *reinterpret_cast<const floatx4 *>(p + 4);
    }
    __device__ __forceinline__ float get(int i) const { return i < 4 ? a[i & 3] : b[i & 3]; }
    static __device__ __forceinline__ void store(float *p, const float (&f)[8])
    {
        *reinterpret_cast<floatx4 *>(p) = floatx4{f[0], f[1], f[2], f[3]};
        *reinterpret_cast<floatx4 *>(p + 4) = floatx4{f[4], f[5], f[6], f[7]};
    }
};

template <typename IO, int NP> struct MergeRow {
    const float *oc;   // o_comp of the row, or null: out = o_sel
    const IO *gate;    // of the row, or null: g = 1/2
    Io8<float> c[NP];
    Io8<IO> gl[NP];

    // channel(j): the first of the lane's eight channels of pair j
    template <typename Channel> __device__ __forceinline__ void load(const float *oc_row, const IO *gate_row, Channel &&channel)
    {
        oc = oc_row;
        gate = gate_row;
        if (oc != nullptr) {
#pragma unroll
            for (int j = 0; j < NP; ++j) c[j].load(oc + channel(j));
            if (gate != nullptr) {
#pragma unroll
                for (int j = 0; j < NP; ++j) gl[j].load(gate + channel(j));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // os[j]: o_sel in these channels
    template <typename Channel>
    __device__ __forceinline__ void store(const float (&os)[NP][8], IO *out_row, IO *o_sel_row, Channel &&channel)
    {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            float res[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) res[i] = os[j][i];
            if (oc != nullptr) {
                float gt[8] = {0.5f, 0.5f, 0.5f, 0.5f, 0.5f, 0.5f, 0.5f, 0.5f};
                if (gate != nullptr) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) gt[i] = 1.f / (1.f + __expf(-gl[j].get(i)));
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) res[i] = gt[i] * c[j].get(i) + (1.f - gt[i]) * os[j][i];
            }
            Io8<IO>::store(out_row + channel(j), res);
            if (o_sel_row != nullptr) Io8<IO>::store(o_sel_row + channel(j), os[j]);
        }
    }
};

// Runs a and b of a 32x32 MFMA's accumulators, four registers each: the lane's rows 8 r + 4 g .. + 3 and 8 (r + 1) + 4 g .. + 3
// (g = lane / 32) -> rows 8 (r + g) .. + 7.
__device__ __forceinline__ void join_runs_32(const float (&a)[4], const float (&b)[4], float (&o)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[e]), __float_as_uint(b[e]), false, false);
        o[e] = __uint_as_float(x[0]);
        o[4 + e] = __uint_as_float(x[1]);
    }
}

// The same for two 16x16 tiles, rows 4 g .. + 3 of either (g = lane / 16): rows 8 (g / 2) .. + 7 of tile g % 2.
__device__ __forceinline__ void join_runs_16(const float (&a)[4], const float (&b)[4], float (&o)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[e]), __float_as_uint(b[e]), false, false);
        o[e] = __uint_as_float(x[0]);
        o[4 + e] = __uint_as_float(x[1]);
    }
}

// Work mapping of the selection kernels: workgroup id mod 8 is its XCD, and each XCD has an L2 of its own.  Neighbouring
// query blocks share key blocks, so an XCD works on neighbours: on a contiguous eighth of every head's query blocks, all
// XCDs on the same head at a time, or (whole_heads) on a contiguous eighth of all (head, query block) pairs.
// The former keeps the key blocks in use together in the memory-side cache (1000 views: 43.9 ms, 52.5 the other way; 300
// views, blocks of 128: 18.7 and 21.0); the latter lets an XCD read few heads only, which pays where a head's K and V fit
// an L2 or two of 4 MiB (16 heads, blocks of 64, microseconds, former -> latter: 4 views 65.9 -> 63.5, 8 views 108.5 ->
// 102, 12: 157.5 -> 153, 16: 200.6 -> 195.5, 24 views (8.4 MB a head) 322 -> 321, 40: 764 -> 763, 100: 2055 -> 2127; blocks of
// 32, 8 views 127.3 -> 120, 20 views (7 MB) 334 -> 325; fp32, 8 views (7 MB) 247 -> 242, 16 views 514 -> 515).
constexpr int64_t kWholeHeadBytes = int64_t(8) << 20;

inline bool xcd_whole_heads(const SelectArgs &a)
{
    return a.n_blk * a.block * 64 * 2 * (a.is_bf16 ? 2 : 5) <= kWholeHeadBytes;  // fp32: three parts of K, two of V
}

inline int64_t xcd_grid(int64_t n_sets, int heads, bool whole_heads)
{
    return whole_heads ? (n_sets * heads + 7) / 8 * 8 : (n_sets + 7) / 8 * 8 * heads;
}

// Head and set of workgroup `bid`; false: none.
__device__ __forceinline__ bool xcd_item(int64_t bid, int64_t n_sets, int heads, bool whole_heads, int &h, int64_t &set)
{
    if (whole_heads) {
        const int64_t per = (n_sets * heads + 7) / 8, item = (bid & 7) * per + (bid >> 3);
        h = static_cast<int>(item / n_sets);
        set = item - h * n_sets;
        return h < heads;
    }
    const int64_t per = (n_sets + 7) / 8;
    h = static_cast<int>(bid / (8 * per));
    const int64_t r = bid % (8 * per);
    set = (r % 8) * per + r / 8;
    return set < n_sets;
}

}  // namespace s3r
