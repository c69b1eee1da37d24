// What the attention kernels share: constants of the weights' arithmetic, tile copies into LDS, maxima that carry NaN.
#pragma once
#include "sla_common.hpp"

namespace sla {

constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((address_space(3))) void *lds_void_p;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

// XOR swizzle of 16-byte chunks: 8 chunks per 128-byte row / 4 chunks per 64-byte row
__device__ __forceinline__ int swz8(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int swz4(int row) { return (row >> 2) & 3; }

// Waits until this wave's tile copies have landed and its LDS reads have returned, then joins the workgroup.  The copies are issued from inline assembly so that the compiler's own wait-count
// insertion does not see them: it would otherwise drain ALL outstanding copies (vmcnt(0)) before every LDS read
// and serialise the prefetch ring.  The waits are therefore explicit.
__device__ __forceinline__ void wait_copies_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint32_t pack_f16(float lo, float hi)
{
    f16x2 r;
    r[0] = (_Float16)lo;
    r[1] = (_Float16)hi;
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ f16x8 pack8_f16(const f32x16 &a, int base)
{
    uint4 o;
    o.x = pack_f16(a[base + 0], a[base + 1]); o.y = pack_f16(a[base + 2], a[base + 3]);
    o.z = pack_f16(a[base + 4], a[base + 5]); o.w = pack_f16(a[base + 6], a[base + 7]);
    return __builtin_bit_cast(f16x8, o);
}
// Largest of the 16 values a lane holds of one unit of S^T, and over the lane pair that shares the row: NaN if one of them is (v_maximum3_f32)
__device__ __forceinline__ float max3_nan(float a, float b, float c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); }
__device__ __forceinline__ float max16_nan(const f32x16 &s)
{
    const float a = max3_nan(s[0], s[1], s[2]), b = max3_nan(s[3], s[4], s[5]), c = max3_nan(s[6], s[7], s[8]);
    const float d = max3_nan(s[9], s[10], s[11]), e = max3_nan(s[12], s[13], s[14]);
    return max3_nan(max3_nan(a, b, c), max3_nan(d, e, s[15]), a);
}
__device__ __forceinline__ float pair_max_nan(float v)
{
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// log2 of the V scale of a lane's list entry relative to the list's reference: the scale of the first entry that has one, or, if a finite
// scale of this window lies more than 2^kFarV above that, the largest of them (first: set it from this window).  A block of zeros
// (lv = -inf) fits any scale and takes the reference.  A block further than 2^kFarV below the reference counts as that far below:
// its values vanish beside the reference's either way, and its weights, with the scale and without, keep within the range of fp32.
constexpr float kFarV = 100.0f;
__device__ __forceinline__ float relative_scale(float lv, bool in, bool first, float &lv_ref)
{
    if (first) {
        const unsigned long long m = __ballot(in && lv != -INFINITY);
        lv_ref = m ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lv), __builtin_ctzll(m))) : 0.f;
    }
    float d = lv == -INFINITY ? 0.f : lv - lv_ref;
    if (__ballot(in && fabsf(d) > kFarV)) {
        const bool above = first && in && lv < INFINITY && d > kFarV;
        if (__ballot(above)) {
            lv_ref = wave_max_dpp(above ? lv : -INFINITY);
            d = lv == -INFINITY ? 0.f : lv - lv_ref;
        }
        d = d < -kFarV ? -kFarV : d;
    }
    return d;
}

// The lane index, computed here (two instructions) and not carried in a register from the top of the kernel
__device__ __forceinline__ int lane_now()
{
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}

// What both attention kernels take (grid: one workgroup per query block, of two waves, or four in attend_kernel<., 2, 2>)
typedef void AttendKernel(const void *__restrict__ Qp, const void *__restrict__ Kp, const uint16_t *__restrict__ Vp, const float *__restrict__ lvs,
                          const float *__restrict__ sQ, const float *__restrict__ sK, RowMap rm, const int32_t *__restrict__ crit_idx, int k_c,
                          const uint16_t *__restrict__ Hq, const uint16_t *__restrict__ WT, int proj_per_head, int phi, int H, int N, int Nqb, int Nkb,
                          long total, float c_exp, uint16_t *__restrict__ O, float *__restrict__ O32);
constexpr int kShortList = 2;                          // lists of at most so many blocks go to the short kernel (64-row query blocks)
AttendKernel *attend_short_kernel_for(bool fp8);

}  // namespace sla
