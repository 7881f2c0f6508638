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
