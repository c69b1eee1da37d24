// Per-key-block linear-attention states (Alg. 1 steps 6-8 of the paper restricted to one
// key block; phi = softmax over the head dimension, or the ELU(x)+1 the algorithm prints):
//     h_j = phi(K_j)^T V_j   (64 x 64),   z_j = sum_t phi(K_j,t)   (64)
// written as bf16 hT[j][e][d] = h_j[d][e] (rows 0..63) and hT[j][64][d] = z_j[d].
//
// A workgroup of four waves takes one key block: all load it and stage K (row-major) and V (transposed) in LDS; then wave 0
// adds the block mean of K (fp64, serial: one lane per channel) and z, wave 1 makes V^T for the attention kernel, waves 2 and
// 3 normalise the token rows (half a row per lane), and each wave takes a quarter of the 64x64x64 product on
// v_mfma_f32_32x32x16_bf16; the state leaves in the layout the aggregation GEMM and the attention epilogue read.  V^T of the
// block (fp16, key-permuted) lets the attention kernel fetch both of its tiles as plain 16-byte rows, and the block mean is the
// classifier's, so K is read from HBM once per layer by this kernel instead of twice.
// The fp16 copy of V is exact: bf16 values are first divided by the power of two 2^e of the block's largest
// magnitude (so that any bf16 tensor fits the range of fp16; entries more than 2^24 below the block's maximum
// are the only ones to lose bits), E4M3 codes are taken as they are; the attention kernel gets e, or the base-2
// logarithm of the E4M3 block scale, in `lvs` and folds it into the exponent of its softmax weights (-inf for a block of zeros,
// which has no scale of its own).
// The state and V^T tiles leave through LDS so that every store instruction writes 1 KB of whole rows.  The kernel is bound by
// HBM (16 KB in, 16.6 KB out per block for bf16 inputs) where the launch is long, by the life of a block where it is not.
// Seven blocks are in flight per CU (72 registers per lane; 64 for eight spilt, and cost a fifth).  Against one wave per block
// with the next block's loads in flight (eight blocks and eight waves per CU, each block three times as long): 16 heads x
// 43968 tokens bf16 75 -> 59 us (6.3 TB/s), 32 x 16 x 1374 71 -> 58 us, 16 x 10992 22.6 -> 16.7 us, 6 x 16 x 1374 e4m3
// 21 -> 15 us, 2 x 512 7.2 -> 4.3 us.  A few workgroups past the states grid lay out the projection matrices for the
// attention epilogue (one launch fewer).
#include "sla_common.hpp"
#include "sla_kernels.hpp"

namespace sla {

constexpr int kLdsRow = 72;            // bf16 elements per LDS row (64 + 8 pad: 144 B stride)

// Raw global data of one key block, as loaded: K as 16-byte row chunks, V as 8-byte (bf16) or
// 4-byte (e4m3) pieces of four channels arranged for the register transpose.
template <bool FP8>
struct BlockRegs {
    uint32_t k[FP8 ? 4 : 8];     // plain dwords: arrays of vectors are not reliably kept in registers
    uint32_t v[FP8 ? 4 : 8];
};

// Rows past the end of the sequence (ragged last block of a head) repeat the last valid row: their
// phi is multiplied by zero below, and finite stand-in values keep every product finite.
template <bool FP8>
__device__ __forceinline__ void load_block(BlockRegs<FP8> &r, const void *K, const void *V, size_t tok0, int ts, int valid, int tid)
{
    const int last = valid - 1;
    const int eq = tid & 15, tg = tid >> 4;                                      // V: 4 channels (quad eq) x 4 consecutive tokens (group tg)
    if (!FP8) {
        const uint16_t *Kg = (const uint16_t *)K + tok0, *Vg = (const uint16_t *)V + tok0;
        // K: chunk c = tid + 256 x is 8 channels (16 B) of row c/8
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int c = tid + 256 * x, t = min(c >> 3, last), col = (c & 7) * 8;
            const uint4 w = *(const uint4 *)(Kg + (size_t)t * ts + col);
            r.k[4 * x] = w.x; r.k[4 * x + 1] = w.y; r.k[4 * x + 2] = w.z; r.k[4 * x + 3] = w.w;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = min(tg * 4 + k, last);
            const uint2 w = *(const uint2 *)(Vg + (size_t)t * ts + 4 * eq);
            r.v[2 * k] = w.x;
            r.v[2 * k + 1] = w.y;
        }
    } else {
        const uint8_t *Kg = (const uint8_t *)K + tok0, *Vg = (const uint8_t *)V + tok0;
        // K: chunk c = tid is 16 channels (16 B of e4m3) of row c/4
        const uint4 w = *(const uint4 *)(Kg + (size_t)min(tid >> 2, last) * ts + (tid & 3) * 16);
        r.k[0] = w.x; r.k[1] = w.y; r.k[2] = w.z; r.k[3] = w.w;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = min(tg * 4 + k, last);
            r.v[k] = *(const uint32_t *)(Vg + (size_t)t * ts + 4 * eq);
        }
    }
}

__device__ __forceinline__ uint4 e4m3x8_to_bf16x8(uint32_t lo, uint32_t hi)
{
    const f32x2 a0 = __builtin_amdgcn_cvt_pk_f32_fp8(lo, false), a1 = __builtin_amdgcn_cvt_pk_f32_fp8(lo, true);
    const f32x2 a2 = __builtin_amdgcn_cvt_pk_f32_fp8(hi, false), a3 = __builtin_amdgcn_cvt_pk_f32_fp8(hi, true);
    uint4 o;
    o.x = pack_bf16(a0[0], a0[1]); o.y = pack_bf16(a1[0], a1[1]);
    o.z = pack_bf16(a2[0], a2[1]); o.w = pack_bf16(a3[0], a3[1]);
    return o;
}

// Largest magnitude bits among the bf16 values of V that a wave holds for one key block.
__device__ __forceinline__ uint32_t wave_max_magnitude(const uint32_t (&v)[8])
{
    uint32_t mx = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) mx = max(mx, max(v[x] & 0x7FFFu, (v[x] >> 16) & 0x7FFFu));
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
    return mx;
}

// four bf16 (two dwords) times 2^sh -> four fp16 (two dwords), round to nearest even where bits are lost
__device__ __forceinline__ uint2 bf16x4_to_f16x4(uint2 w, int sh)
{
    typedef __attribute__((ext_vector_type(2))) _Float16 h2;
    h2 a, b;
    a[0] = (_Float16)ldexpf(bf16_lo(w.x), sh); a[1] = (_Float16)ldexpf(bf16_hi(w.x), sh);
    b[0] = (_Float16)ldexpf(bf16_lo(w.y), sh); b[1] = (_Float16)ldexpf(bf16_hi(w.y), sh);
    return make_uint2(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b));
}

// Registers -> LDS: K rows as bf16 (e4m3 codes widened exactly, the block scale is applied later
// in fp32), V transposed to [channel][token] bf16 (e4m3 widened exactly, unscaled).
template <bool FP8>
__device__ __forceinline__ void stage_block(const BlockRegs<FP8> &r, uint16_t *Ks, uint16_t *Vt, int tid)
{
    const int eq = tid & 15, tg = tid >> 4;
    uint16_t *dst = Vt + (4 * eq) * kLdsRow + tg * 4;
    const uint32_t *w = r.v;
    if (!FP8) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int c = tid + 256 * x, t = c >> 3, col = (c & 7) * 8;
            *(uint4 *)(Ks + t * kLdsRow + col) = make_uint4(r.k[4 * x], r.k[4 * x + 1], r.k[4 * x + 2], r.k[4 * x + 3]);
        }
        // w[2k], w[2k+1]: channels 4eq .. 4eq+3 of token 4 tg + k -> channel 4eq + c over the 4 tokens
        *(uint2 *)(dst) = make_uint2(__builtin_amdgcn_perm(w[2], w[0], 0x05040100), __builtin_amdgcn_perm(w[6], w[4], 0x05040100));
        *(uint2 *)(dst + kLdsRow) = make_uint2(__builtin_amdgcn_perm(w[2], w[0], 0x07060302), __builtin_amdgcn_perm(w[6], w[4], 0x07060302));
        *(uint2 *)(dst + 2 * kLdsRow) = make_uint2(__builtin_amdgcn_perm(w[3], w[1], 0x05040100), __builtin_amdgcn_perm(w[7], w[5], 0x05040100));
        *(uint2 *)(dst + 3 * kLdsRow) = make_uint2(__builtin_amdgcn_perm(w[3], w[1], 0x07060302), __builtin_amdgcn_perm(w[7], w[5], 0x07060302));
    } else {
        const int t = tid >> 2, col = (tid & 3) * 16;
        *(uint4 *)(Ks + t * kLdsRow + col) = e4m3x8_to_bf16x8(r.k[0], r.k[1]);
        *(uint4 *)(Ks + t * kLdsRow + col + 8) = e4m3x8_to_bf16x8(r.k[2], r.k[3]);
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            float f[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f32x2 p = (ch & 2) ? __builtin_amdgcn_cvt_pk_f32_fp8(w[k], true) : __builtin_amdgcn_cvt_pk_f32_fp8(w[k], false);
                f[k] = p[ch & 1];
            }
            *(uint2 *)(dst + ch * kLdsRow) = make_uint2(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]));
        }
    }
}

template <bool FP8>
__global__ __launch_bounds__(256, 7) void states_kernel(const void *__restrict__ K, const void *__restrict__ V,
                                                                  const float *__restrict__ sK, const float *__restrict__ sV,
                                                                  RowMap rm, int N, int Nkb,
                                                                  uint16_t *__restrict__ hT, uint16_t *__restrict__ Vp, float *__restrict__ lvs,
                                                                  double *__restrict__ kbar, int phi, unsigned first, unsigned state_wgs,
                                                                  const uint16_t *__restrict__ W, uint16_t *__restrict__ WT)
{
    asm volatile("" ::"s"(K), "s"(V), "s"(sK), "s"(sV), "s"(rm.bs), "s"(rm.hs), "s"(rm.ts), "s"(rm.H), "s"(N), "s"(Nkb), "s"(hT), "s"(Vp), "s"(lvs), "s"(kbar), "s"(phi), "s"(first), "s"(state_wgs), "s"(W), "s"(WT));      // all kernel arguments in one batch of scalar loads, here
    if (blockIdx.x >= state_wgs) {     // workgroups past the states grid each lay out one projection matrix for the attention kernel
        const size_t m = (size_t)(blockIdx.x - state_wgs) * kD * kD;
        transpose_w_tile(W + m, WT + m, 256);
        return;
    }
    __shared__ __attribute__((aligned(16))) uint16_t Ks[64 * kLdsRow];           // K rows, later phi^T [d][t], later the state
    __shared__ __attribute__((aligned(16))) uint16_t Vt[64 * kLdsRow];           // V^T [e][t]
    __shared__ uint32_t vmag[4];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, g = lane >> 5;
    const long blk = first + blockIdx.x, bh = (long)((unsigned)blk / (unsigned)Nkb);
    const int t0 = (int)(blk - bh * Nkb) * kBK, valid = min(kBK, N - t0);
    {
        BlockRegs<FP8> regs;
        load_block<FP8>(regs, K, V, rm.head(bh) + (size_t)t0 * rm.ts, rm.ts, valid, tid);
        stage_block<FP8>(regs, Ks, Vt, tid);
        uint32_t mx;
        if constexpr (FP8) mx = __ballot(((regs.v[0] | regs.v[1] | regs.v[2] | regs.v[3]) & 0x7F7F7F7Fu) != 0u) != 0ull;   // zero or not is all there is to know
        else mx = wave_max_magnitude(regs.v);
        if (lane == 0) vmag[wave] = mx;
    }
    lds_barrier();
    const uint32_t vmax = max(max(vmag[0], vmag[1]), max(vmag[2], vmag[3]));     // bits of the block's largest |V| (e4m3: 0 or 1)
    const int vexp = FP8 ? 127 : min(max((int)(vmax >> 7), 1), 254);             // its exponent field (127 = 2^0)

    uint32_t xp[16];                             // phi of the lane's half row, bf16 pairs
    if (wave == 0) {
        // ---- block mean of K for the classifier: lane d adds the tokens of channel d serially in fp64
        // (ascending token order) and multiplies by 1/count -- the same arithmetic as the pooling kernel
        if (kbar != nullptr) {
            const double s = FP8 ? (double)sK[blk] : 1.0;
            double acc = 0.0;
            auto add = [&](int t) {
                const double v = (double)bf16_bits_to_f32(Ks[t * kLdsRow + lane]);
                acc += FP8 ? v * s : v;
            };
            if (valid == kBK) {
#pragma unroll 16
                for (int t = 0; t < kBK; ++t) add(t);
            } else {
                for (int t = 0; t < valid; ++t) add(t);
            }
            kbar[blk * kD + lane] = acc * (1.0 / (double)valid);
        }
    } else if (wave >= 2) {
        // ---- phi: lane (l32, g) of wave 2, 3 owns channels 32 g .. of token row 32 (wave - 2) + l32; the other half row is
        // the lane's 32 positions away
        float x[32];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint4 w = *(const uint4 *)(Ks + (32 * (wave - 2) + l32) * kLdsRow + 32 * g + c * 8);
            x[c * 8 + 0] = bf16_lo(w.x); x[c * 8 + 1] = bf16_hi(w.x);
            x[c * 8 + 2] = bf16_lo(w.y); x[c * 8 + 3] = bf16_hi(w.y);
            x[c * 8 + 4] = bf16_lo(w.z); x[c * 8 + 5] = bf16_hi(w.z);
            x[c * 8 + 6] = bf16_lo(w.w); x[c * 8 + 7] = bf16_hi(w.w);
        }
        // phi = 0: softmax over the 64 channels; phi = 1: ELU(x)+1 elementwise (x+1 above 0, exp(x) below).
        // s is 1 for bf16 inputs and the K block scale for e4m3.
        const bool real = 32 * (wave - 2) + l32 < valid;         // rows past the sequence end contribute nothing
        const float cexp = (FP8 ? sK[blk] : 1.0f) * 1.4426950408889634f;
        float inv;
        if (phi == 0) {
            float mx = x[0];
#pragma unroll
            for (int d = 1; d < 32; ++d) mx = fmaxf(mx, x[d]);
            mx = pair_max(mx);
            // exp(s*(x - mx)) = exp2(x*c - mx*c), c = s*log2(e)
            const float mc = mx * cexp;
            float sum = 0.f;
#pragma unroll
            for (int d = 0; d < 32; ++d) {
                x[d] = fast_exp2(fmaf(x[d], cexp, -mc));
                sum += x[d];
                if ((d & 7) == 7) __builtin_amdgcn_sched_barrier(0);         // (all arguments formed ahead of the exponentials spilt registers)
            }
            sum += xchg32(sum);
            inv = real ? 1.0f / sum : 0.0f;
        } else {
            const float sc = FP8 ? sK[blk] : 1.0f;
#pragma unroll
            for (int d = 0; d < 32; ++d) {
                x[d] = x[d] > 0.f ? fmaf(x[d], sc, 1.0f) : fast_exp2(x[d] * cexp);
                if ((d & 7) == 7) __builtin_amdgcn_sched_barrier(0);
            }
            inv = real ? 1.0f : 0.0f;
        }
#pragma unroll
        for (int d = 0; d < 16; ++d) xp[d] = pack_bf16(x[2 * d] * inv, x[2 * d + 1] * inv);
    } else if (Vp != nullptr) {
        // ---- V^T tile for the attention kernel: Vp[e][.] with the 2nd and 3rd group of 4 tokens of every
        // 16 swapped (slot 16s + 8g + 4a + b holds token 16s + 8a + 4g + b), which is the key order the
        // accumulator-as-operand trick of that kernel needs.  fp16: bf16 V divided by 2^(vexp - 127), e4m3 codes as they are.
        uint16_t *vt = Vp + (size_t)blk * kD * kBK;
        const int c = lane & 7, src = 16 * (c >> 1) + 4 * (c & 1);   // 16-byte piece c of a row: tokens src..src+3, src+8..src+11
#pragma unroll
        for (int x8 = 0; x8 < 8; ++x8) {                             // a wave-wide store covers 8 whole rows (1 KB)
            const int e = 8 * x8 + (lane >> 3);
            const uint2 lo = bf16x4_to_f16x4(*(const uint2 *)(Vt + e * kLdsRow + src), 127 - vexp);
            const uint2 hi = bf16x4_to_f16x4(*(const uint2 *)(Vt + e * kLdsRow + src + 8), 127 - vexp);
            *(uint4 *)(vt + e * kBK + 8 * c) = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        if (lane == 0) lvs[blk] = vmax == 0u ? -INFINITY : FP8 ? __log2f(fmaxf(sV[blk], 1e-30f)) : (float)(vexp - 127);
    }
    lds_barrier();                                          // the rows are in registers and added: Ks may be overwritten
    if (wave >= 2) {
        uint16_t *col = Ks + 32 * g * kLdsRow + 32 * (wave - 2) + l32;
#pragma unroll
        for (int d = 0; d < 16; ++d) {
            col[(2 * d) * kLdsRow] = (uint16_t)(xp[d] & 0xFFFFu);
            col[(2 * d + 1) * kLdsRow] = (uint16_t)(xp[d] >> 16);
        }
    }
    lds_barrier();

    // ---- h[d][e] = sum_t phi^T[d][t] * V^T[e][t]: wave w takes d = 32 (w / 2) .., e = 32 (w % 2) ..
    const int da = 32 * (wave >> 1), eb = 32 * (wave & 1);
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const bf16x8 af = *(const bf16x8 *)(Ks + (da + l32) * kLdsRow + 16 * s + 8 * g);
        const bf16x8 bfr = *(const bf16x8 *)(Vt + (eb + l32) * kLdsRow + 16 * s + 8 * g);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc, 0, 0, 0);
    }
    uint16_t *out = hT + (size_t)blk * kStateElems;
    // ---- z: lane d sums phi^T row d (the bf16 values the product consumes)
    if (wave == 0) {
        constexpr uint32_t kOnes = 0x3F803F80u;             // two bf16 1.0: a dot product with them adds a pair of values
        float z0 = 0.f, z1 = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint4 w = *(const uint4 *)(Ks + lane * kLdsRow + c * 8);
            z0 = dot2_bf16(w.z, kOnes, dot2_bf16(w.x, kOnes, z0));
            z1 = dot2_bf16(w.w, kOnes, dot2_bf16(w.y, kOnes, z1));
        }
        out[64 * kD + lane] = (uint16_t)(pack_bf16(z0 + z1, 0.f) & 0xFFFFu);
    }

    // ---- write hT[e][d]: accumulator register 4q+r holds d = da + 8q + 4g + r, e = eb + l32.
    // The tile goes through LDS (phi^T is consumed) so that it leaves as whole rows, 1 KB per wave-wide store.
    const float vs = FP8 ? sV[blk] : 1.0f;
    lds_barrier();                                          // the operand reads of phi^T are done
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *(uint2 *)(Ks + (eb + l32) * kLdsRow + da + 8 * q + 4 * g) = make_uint2(pack_bf16(acc[4 * q + 0] * vs, acc[4 * q + 1] * vs), pack_bf16(acc[4 * q + 2] * vs, acc[4 * q + 3] * vs));
    lds_barrier();
#pragma unroll
    for (int x2 = 0; x2 < 2; ++x2) {
        const int e = 16 * wave + 8 * x2 + (lane >> 3), c = lane & 7;
        *(uint4 *)(out + e * kD + 8 * c) = *(const uint4 *)(Ks + e * kLdsRow + 8 * c);
    }
}

hipError_t launch_states(const void *K, const void *V, const float *sK, const float *sV, bool fp8, RowMap rm,
                         int BH, int N, void *hT, void *Vp, float *lvs, double *kbar, int phi, const void *W, int nW, void *WT, hipStream_t st)
{
    const int Nkb = (N + kBK - 1) / kBK;
    const long nblocks = (long)BH * Nkb;
    // a launch takes at most 2^20 blocks (a grid is limited to 2^32 threads; 2^20 blocks are some 6 ms); the last one lays out W
    constexpr long kMost = 1l << 20;
    for (long first = 0; first < nblocks; first += kMost) {
        const bool last = nblocks - first <= kMost;
        const unsigned grid = (unsigned)(last ? nblocks - first : kMost), extra = last && W != nullptr ? (unsigned)nW : 0u;
        if (fp8) states_kernel<true><<<grid + extra, 256, 0, st>>>(K, V, sK, sV, rm, N, Nkb, (uint16_t *)hT, (uint16_t *)Vp, lvs, kbar, phi, (unsigned)first, grid, (const uint16_t *)W, (uint16_t *)WT);
        else     states_kernel<false><<<grid + extra, 256, 0, st>>>(K, V, sK, sV, rm, N, Nkb, (uint16_t *)hT, (uint16_t *)Vp, lvs, kbar, phi, (unsigned)first, grid, (const uint16_t *)W, (uint16_t *)WT);
    }
    return hipGetLastError();
}

}  // namespace sla
