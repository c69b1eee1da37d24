// attend_kernel's computation (k_attend.hip) for SHORT critical lists (frame attention: one or two blocks per row; up to kShortList), where
// a workgroup's life is memory latency (list -> tiles, operands of the linear branch) and little arithmetic: no software
// pipeline and no rings, so that the kernel fits 128 registers and 17 KB of LDS and eight workgroups of two waves
// share a CU and hide each other's round trips.  Order of work: the linear branch first (its operands, the Hq^T
// tile, W^T and Z, are asked for together with Q and the list; its result waits in sixteen registers as bf16), then one
// tile at a time through a single K slot and a single V^T slot: S^T, exact running maximum, fp16 weights carrying the
// block's V exponent, O^T += V^T P^T; at the end O = O_sparse / l + O_lin W.
// What bounds it: the bytes (Q, K, V^T, Hq in, O out; 453 MB on 32 frames of 16 heads x 1374 tokens: 96 us, 4.7 TB/s).  102 us before
// the vector work per unit was cut: no key mask but in a ragged block, the V scale in the exponent instead of a product per weight,
// no rescale of empty accumulators (6 E4M3 frames 23.4 -> 21.5 us).
// (Two tile buffers, the copies of tile c+1 in flight while tile c is worked on, were measured on lists of nine: a
// workgroup then lives 20 us instead of 31, but only four fit a CU instead of eight, and the launch takes the same time.)
#include "attend_common.hpp"
#include "sla_kernels.hpp"

namespace sla {

// Two copies of 1 KB, from base0 + v0 and base1 + v1, to consecutive kilobytes of LDS in one statement
__device__ __forceinline__ void copy_2k_to_lds(const uint8_t *base0, const uint8_t *base1, uint32_t v0, uint32_t v1, uint32_t lds_addr)
{
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "v"(v0), "v"(v1), "s"(base0), "s"(base1), "s"(lds_addr) : "memory", "scc");
}
// N such copies (an even number) of consecutive 1 KB pieces of a tile: piece x starts at base + x stride in memory and takes the per-lane
// offset voff, for odd x with bit 6 flipped if FLIP (see CopyOffsets)
template <int N, bool FLIP> __device__ __forceinline__ void copy_nk_to_lds(const uint8_t *base, uint32_t stride, uint32_t voff, uint32_t lds_addr)
{
    static_assert(N % 2 == 0, "pieces go in pairs");
    const uint32_t odd = FLIP ? voff ^ 64u : voff;
#pragma unroll
    for (int x = 0; x < N; x += 2) copy_2k_to_lds(base + x * stride, base + (x + 1) * stride, voff, odd, lds_addr + x * 1024);
}

// The row sums are those of the weights with the V scale 2^lsv, divided by it, unless it is further than 2^kFarSum from the list's
// reference: fp32 holds a scaled weight down to 2^-126 of the largest, one that counts in the sum (2^-30 of it) down to a scale of 2^-96.
constexpr float kFarSum = 32.0f;

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
// largest of the 16 values a lane holds of one unit of S^T
__device__ __forceinline__ float max16(const f32x16 &s)
{
    const float a = max3(s[0], s[1], s[2]), b = max3(s[3], s[4], s[5]), c = max3(s[6], s[7], s[8]);
    const float d = max3(s[9], s[10], s[11]), e = max3(s[12], s[13], s[14]);
    return max3(max3(a, b, c), max3(d, e, s[15]), a);
}

constexpr int kWaves = 2;                              // of 32 query rows
template <bool FP8>
struct Tile {
    static constexpr int KBYTES = FP8 ? 64 * 64 : 64 * 128;     // K tile (e4m3 / bf16)
    static constexpr int VBYTES = 64 * 128;                     // V^T tile (always fp16)
    static constexpr int KINS = KBYTES / 1024 / kWaves;         // 1 KB copy instructions per wave
    static constexpr int VINS = VBYTES / 1024 / kWaves;
};

// Per-lane byte offset of the 16-byte chunk each lane copies in one 1 KB instruction: LDS position (row, slot) <- global
// chunk slot ^ swizzle(row).  Instruction `ins` of a tile covers rows 8 ins .. (128-byte rows) or 16 ins .. (64-byte rows),
// which advances the swizzle by 4 ins mod 8 (a flip of offset bit 6 for odd ins) or by 4 ins mod 4 = 0: one register
// serves all of a wave's copies, the rows themselves are advanced in the scalar base (row pitches are multiples of 128 bytes
// where the flip is used).
template <bool FP8>
struct CopyOffsets {
    using T = Tile<FP8>;
    static constexpr int kRows = FP8 ? 16 : 8;         // K rows per instruction
    uint32_t k, v;
    uint32_t kstride;                                  // bytes from one K instruction's rows to the next's (uniform)
    int wave_k, wave_v;                                // first instruction of this wave (uniform)
    // krowb: bytes between consecutive K rows in global memory (64 or 128 when the heads are contiguous)
    __device__ __forceinline__ void init(int wave_u, int lane, int krowb)
    {
        wave_k = wave_u * T::KINS;
        wave_v = wave_u * T::VINS;
        kstride = (uint32_t)kRows * (uint32_t)krowb;
        const uint32_t r = lane >> 3, chunk = (uint32_t)((lane & 7) ^ swz8(r)) << 4;
        v = r * 128u + chunk;
        k = FP8 ? (uint32_t)(lane >> 2) * (uint32_t)krowb + ((uint32_t)((lane & 3) ^ swz4(lane >> 2)) << 4) : r * (uint32_t)krowb + chunk;
    }
    // this wave's share of the K tile at kt / of a contiguous 8 KB tile at vt, to the tile at LDS address dst
    __device__ __forceinline__ void copy_k(const uint8_t *kt, uint32_t dst) const
    {
        copy_nk_to_lds<T::KINS, !FP8>(kt + wave_k * kstride, kstride, k, dst + wave_k * 1024);
    }
    __device__ __forceinline__ void copy_v(const uint8_t *vt, uint32_t dst) const
    {
        copy_nk_to_lds<T::VINS, true>(vt + wave_v * 1024, 1024u, v, dst + wave_v * 1024);
    }
    // the K tile of the ragged last block: rows past the end are clamped to the last one (they are masked later)
    __device__ __forceinline__ void copy_k_ragged(const uint8_t *kt, uint32_t dst, int rows, int krowb) const
    {
        const int lane = lane_now();
#pragma unroll
        for (int x = 0; x < T::KINS; ++x) {
            const int row = (wave_k + x) * kRows + (lane >> (FP8 ? 2 : 3));
            // (offsets from the tile's first row: a lane offset is unsigned, the clamped row may lie before this instruction's first)
            const uint32_t off = (k ^ ((!FP8 && (x & 1)) ? 64u : 0u)) + (uint32_t)((wave_k + x) * (int)kstride - (row - min(row, rows - 1)) * krowb);
            copy_1k_to_lds(kt, off, dst + (wave_k + x) * 1024);
        }
    }
};

template <bool FP8>
__global__ __launch_bounds__(64 * kWaves, 4) void attend_short_kernel(
    const void *__restrict__ Qp, const void *__restrict__ Kp, const uint16_t *__restrict__ Vp, const float *__restrict__ lvs,
    const float *__restrict__ sQ, const float *__restrict__ sK, RowMap rm,
    const int32_t *__restrict__ crit_idx, int k_c, const uint16_t *__restrict__ Hq, const uint16_t *__restrict__ WT,
    int proj_per_head, int phi, int H, int N, int Nqb, int Nkb, long total, float c_exp, uint16_t *__restrict__ O, float *__restrict__ O32)
{
    constexpr int BQ = 32 * kWaves;
    constexpr int ES = FP8 ? 1 : 2;
    constexpr int KROWB = FP8 ? 64 : 128;
    constexpr int kA = 0, kB = 8192, kZ = 16384;      // LDS: slot A (K tile / Hq^T), slot B (V^T tile / W^T), the Z row
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kZ + 256];
    asm volatile("" ::"s"(Qp), "s"(Kp), "s"(Vp), "s"(lvs), "s"(sQ), "s"(sK), "s"(rm.bs), "s"(rm.hs), "s"(rm.ts), "s"(rm.H), "s"(crit_idx),
                 "s"(k_c), "s"(Hq), "s"(WT), "s"(proj_per_head), "s"(phi), "s"(H), "s"(N), "s"(Nqb), "s"(Nkb), "s"(total), "s"(c_exp), "s"(O), "s"(O32));
    const long work = xcd_remap(blockIdx.x, total);
    if (work >= total) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const long bh = (long)((unsigned)work / (unsigned)Nqb);
    const int i = (int)(work - bh * Nqb);
    const int q = i * BQ + 32 * wave + l32;
    const bool qok = q < N;
    const size_t head = rm.head(bh);
    const int krowb = rm.ts * ES;
    const uint8_t *Kh = (const uint8_t *)Kp + head * ES;
    const uint8_t *Vh = (const uint8_t *)(Vp + (size_t)bh * Nkb * kBK * kD);

    // the list (at most kShortList entries, one per lane), then Q
    const int j0 = lane < k_c ? crit_idx[work * (long)k_c + lane] : -1;
    bf16x8 qf[4];
    i32x8 q8;
    if (FP8) {
        uint4 w0 = make_uint4(0, 0, 0, 0), w1 = w0;
        if (qok) {
            const uint8_t *qr = (const uint8_t *)Qp + head + (size_t)q * rm.ts + 32 * g;
            w0 = *(const uint4 *)qr;
            w1 = *(const uint4 *)(qr + 16);
        }
        q8[0] = w0.x; q8[1] = w0.y; q8[2] = w0.z; q8[3] = w0.w; q8[4] = w1.x; q8[5] = w1.y; q8[6] = w1.z; q8[7] = w1.w;
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            uint4 w = make_uint4(0, 0, 0, 0);
            if (qok) w = *(const uint4 *)((const uint16_t *)Qp + head + (size_t)q * rm.ts + 16 * s + 8 * g);
            qf[s] = __builtin_bit_cast(bf16x8, w);
        }
    }
    const float qscale = FP8 ? sQ[work] : 1.0f;

    CopyOffsets<FP8> co;
    co.init(__builtin_amdgcn_readfirstlane(wave), lane, krowb);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_p)lds;
    const uint32_t ktile_bytes = (uint32_t)kBK * (uint32_t)krowb;
    const int tail_rows = N & (kBK - 1), ragged_j = tail_rows ? Nkb - 1 : -1;

    // ---- the linear branch: operands on their way while the list and Q arrive
    if (Hq != nullptr) {
        const uint8_t *Hi8 = (const uint8_t *)(Hq + (size_t)work * kStateElems);
        const uint8_t *Wh8 = (const uint8_t *)(WT + (proj_per_head ? (size_t)((unsigned)bh % (unsigned)H) * kD * kD : 0));
        co.copy_v(Hi8, lds_base + kA);
        co.copy_v(Wh8, lds_base + kB);
        if (tid < 8) copy_1k_to_lds(Hi8 + 64 * kD * 2, tid * 16, lds_base + kZ);
    }
    // number of leading valid entries, their V exponents and exp2 constants (a gather that depends on the list)
    const bool jok = j0 >= 0 && j0 < Nkb;
    const unsigned long long okm = __ballot(jok);
    int k = okm == ~0ull ? 64 : __builtin_ctzll(~okm);
    k = __builtin_amdgcn_readfirstlane(min(k, k_c));
    const int d_j = jok ? j0 : 0;
    float lv = lvs[bh * Nkb + d_j];
    float d_cj = FP8 ? fmaxf(c_exp * qscale * sK[bh * Nkb + d_j], 1e-30f) : c_exp;
    asm volatile("" : "+v"(lv), "+v"(d_cj));
    float lv_ref = 0.f;
    const float d_lv = relative_scale(lv, lane < k, true, lv_ref);
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));      // vmcnt(0): Q, the list and the operands have landed
    wait_copies_and_barrier();

    f32x16 zero16;
#pragma unroll
    for (int x = 0; x < 16; ++x) zero16[x] = 0.f;
    uint32_t lin[16];                                  // O_lin W of this lane's row, bf16 pairs (channel 32e + 8a + 4g + b: lin[8e + 2a + b/2])
#pragma unroll
    for (int x = 0; x < 16; ++x) lin[x] = 0u;
    if (Hq != nullptr) {
        const uint8_t *stA = lds + kA, *stB = lds + kB, *zrow = lds + kZ;
        float x[32];
        if (FP8) {
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(q8[w], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(q8[w], true);
                x[4 * w + 0] = lo[0] * qscale; x[4 * w + 1] = lo[1] * qscale; x[4 * w + 2] = hi[0] * qscale; x[4 * w + 3] = hi[1] * qscale;
            }
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint4 w = __builtin_bit_cast(uint4, qf[s]);
                x[8 * s + 0] = bf16_lo(w.x); x[8 * s + 1] = bf16_hi(w.x);
                x[8 * s + 2] = bf16_lo(w.y); x[8 * s + 3] = bf16_hi(w.y);
                x[8 * s + 4] = bf16_lo(w.z); x[8 * s + 5] = bf16_hi(w.z);
                x[8 * s + 6] = bf16_lo(w.w); x[8 * s + 7] = bf16_hi(w.w);
            }
        }
        float inv = 1.0f;
        if (phi == 0) {
            float mx = x[0];
#pragma unroll
            for (int d = 1; d < 32; ++d) mx = fmaxf(mx, x[d]);
            mx = pair_max(mx);
            const float nmx = -mx * kLog2e;
            float sum = 0.f;
#pragma unroll
            for (int d = 0; d < 32; ++d) { x[d] = fast_exp2(fmaf(x[d], kLog2e, nmx)); sum += x[d]; }
            sum += xchg32(sum);
            inv = 1.0f / sum;
        } else {
#pragma unroll
            for (int d = 0; d < 32; ++d) x[d] = x[d] > 0.f ? x[d] + 1.0f : fast_exp2(x[d] * kLog2e);
        }
        bf16x8 fq[4];
        float den = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int dcol = FP8 ? 32 * g + 8 * s : 16 * s + 8 * g;
            uint4 o;
            o.x = pack_bf16(x[8 * s + 0] * inv, x[8 * s + 1] * inv); o.y = pack_bf16(x[8 * s + 2] * inv, x[8 * s + 3] * inv);
            o.z = pack_bf16(x[8 * s + 4] * inv, x[8 * s + 5] * inv); o.w = pack_bf16(x[8 * s + 6] * inv, x[8 * s + 7] * inv);
            fq[s] = __builtin_bit_cast(bf16x8, o);
            const uint4 z = *(const uint4 *)(zrow + dcol * 2);
            den = dot2_bf16(o.w, z.w, dot2_bf16(o.z, z.z, dot2_bf16(o.y, z.y, dot2_bf16(o.x, z.x, den))));
        }
        den += xchg32(den);
        const float inv_den = den > 0.f ? 1.0f / den : 0.f;
        f32x16 lacc[2];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int hchunk = FP8 ? 4 * g + s : 2 * s + g;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const bf16x8 hf = *(const bf16x8 *)(stA + (32 * e + l32) * 128 + ((hchunk ^ swz8(l32)) << 4));
                lacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hf, fq[s], s == 0 ? zero16 : lacc[e], 0, 0, 0);
            }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int y = 0; y < 16; ++y) lacc[e][y] *= inv_den;
        f32x16 pl[2];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bf16x8 pf = pack8(lacc[s >> 1], 8 * (s & 1));
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const bf16x8 wf = *(const bf16x8 *)(stB + (32 * e + l32) * 128 + (((2 * s + g) ^ swz8(l32)) << 4));
                pl[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, pf, s == 0 ? zero16 : pl[e], 0, 0, 0);
            }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int y = 0; y < 8; ++y) lin[8 * e + y] = pack_bf16(pl[e][2 * y], pl[e][2 * y + 1]);
    }
    wait_copies_and_barrier();                      // every wave is done with the operands: the slots take tiles now
    auto request_tile = [&](int c) __attribute__((always_inline)) {
        const uint32_t j = (uint32_t)__builtin_amdgcn_readlane(d_j, c);
        const uint8_t *kt = Kh + (uint64_t)j * ktile_bytes;
        if ((int)j != ragged_j) co.copy_k(kt, lds_base + kA);
        else co.copy_k_ragged(kt, lds_base + kA, tail_rows, krowb);
        co.copy_v(Vh + (uint64_t)j * (uint32_t)(kBK * kD * 2), lds_base + kB);
    };

    // ---- the tiles, one at a time
    int koff[4], voff[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
        koff[s] = FP8 ? l32 * 64 + ((((2 * g + (s & 1)) ^ swz4(l32))) << 4) : l32 * 128 + (((2 * s + g) ^ swz8(l32)) << 4);
#pragma unroll
    for (int st = 0; st < 4; ++st) voff[st] = l32 * 128 + (((2 * st + g) ^ swz8(l32)) << 4);
    f32x16 oacc[2] = {zero16, zero16};
    float m_run = -INFINITY, l_sum = 0.f;
    for (int c = 0; c < k; ++c) {
        const uint8_t *ldsb = lds;
        const uint32_t j = (uint32_t)__builtin_amdgcn_readlane(d_j, c);
        request_tile(c);
        const int valid = (int)j == ragged_j ? tail_rows : kBK;
        const float cj = FP8 ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(d_cj), c)) : c_exp;
        const float lsv = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(d_lv), c));
        const bool far = !(fabsf(lsv) <= kFarSum);     // then the weights are summed without the V scale
        const float per_scale = far ? 0.f : fast_exp2(-lsv);
        wait_copies_and_barrier();                  // tile c has landed
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            f32x16 sacc;
            if (FP8) {
                const i32x4 w0 = *(const i32x4 *)(ldsb + kA + half * 32 * KROWB + koff[0]), w1 = *(const i32x4 *)(ldsb + kA + half * 32 * KROWB + koff[1]);
                i32x8 k8;
                k8[0] = w0[0]; k8[1] = w0[1]; k8[2] = w0[2]; k8[3] = w0[3]; k8[4] = w1[0]; k8[5] = w1[1]; k8[6] = w1[2]; k8[7] = w1[3];
                sacc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(k8, q8, zero16, 0, 0, 0, 0, 0, 0);
            } else {
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const bf16x8 kf = *(const bf16x8 *)(ldsb + kA + half * 32 * KROWB + koff[st]);
                    sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[st], st == 0 ? zero16 : sacc, 0, 0, 0);
                }
            }
            const float top = pair_max(max16(sacc)) * cj + lsv;        // (keys past the end of a ragged block repeat its last one)
            if (c == 0 && half == 0) m_run = fmaxf(m_run, top);        // (nothing to rescale yet)
            else if (__ballot(top > m_run)) {
                const float m_new = fmaxf(m_run, top);
                const float lower = fast_exp2(m_run - m_new), alpha = m_new == m_run ? 1.0f : lower;
                l_sum *= alpha;
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int x = 0; x < 16; ++x) oacc[e][x] *= alpha;
                m_run = m_new;
            }
            const float mfin = m_run == -INFINITY ? 0.f : m_run, moff = lsv - mfin;
            auto real = [&](int x) { return 8 * (x >> 2) + (x & 3) < valid - 32 * half - 4 * g; };      // keys past the end get no weight
            if (far) {
                float plain = 0.f;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const float e = fast_exp2(fmaf(sacc[x], cj, -mfin));
                    plain += real(x) ? e : 0.f;
                }
                l_sum += plain;
            }
            float sum = 0.f;                                           // with the V scale, which is divided out once
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                sacc[x] = fast_exp2(fmaf(sacc[x], cj, moff));
                sum += sacc[x];
            }
            f16x8 p[2] = {pack8_f16(sacc, 0), pack8_f16(sacc, 8)};
            if (valid != kBK) {
                sum = 0.f;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    sum += real(x) ? sacc[x] : 0.f;
                    p[x >> 3][x & 7] = real(x) ? p[x >> 3][x & 7] : (_Float16)0.f;
                }
            }
            l_sum = fmaf(sum, per_scale, l_sum);
#pragma unroll
            for (int ss = 0; ss < 2; ++ss)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const f16x8 vf = *(const f16x8 *)(ldsb + kB + e * 32 * 128 + voff[2 * half + ss]);
                    oacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, p[ss], oacc[e], 0, 0, 0);
                }
        }
        wait_copies_and_barrier();                  // all waves are done with the tile before the next one is asked for
    }

    // ---- O = O_sparse / l + O_lin W
    const float l_run = l_sum + xchg32(l_sum);
    const float inv_l = l_run > 0.f ? fast_exp2(lv_ref) / l_run : l_run;     // 0 for an empty list, NaN for a spoilt row
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            oacc[e][2 * y] = fmaf(oacc[e][2 * y], inv_l, bf16_lo(lin[8 * e + y]));
            oacc[e][2 * y + 1] = fmaf(oacc[e][2 * y + 1], inv_l, bf16_hi(lin[8 * e + y]));
        }
    if (O32 != nullptr) {
        if (qok) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int aa = 0; aa < 4; ++aa)
                    *(float4 *)(O32 + head + (size_t)q * rm.ts + 32 * e + 8 * aa + 4 * g) =
                        make_float4(oacc[e][4 * aa + 0], oacc[e][4 * aa + 1], oacc[e][4 * aa + 2], oacc[e][4 * aa + 3]);
        }
    } else {
        uint8_t *ot = lds + wave * 4096;               // (inside the two slots)
        const int f = ((l32 >> 1) & 7) << 1;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int aa = 0; aa < 4; ++aa) {
                uint2 o;
                o.x = pack_bf16(oacc[e][4 * aa + 0], oacc[e][4 * aa + 1]);
                o.y = pack_bf16(oacc[e][4 * aa + 2], oacc[e][4 * aa + 3]);
                const int piece = 8 * e + 2 * aa + g;
                *(uint2 *)(ot + l32 * 128 + ((piece ^ f) << 3)) = o;
            }
        wave_lds_sync();
        const int q0w = i * BQ + 32 * wave;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int r = 8 * kk + (lane >> 3), ch = lane & 7;
            const int fr = ((r >> 1) & 7) << 1;
            const uint4 v = *(const uint4 *)(ot + r * 128 + (((2 * ch) ^ fr) << 3));
            if (q0w + r < N) *(uint4 *)(O + head + (size_t)(q0w + r) * rm.ts + ch * 8) = v;
        }
    }
}

AttendKernel *attend_short_kernel_for(bool fp8) { return fp8 ? attend_short_kernel<true> : attend_short_kernel<false>; }

}  // namespace sla
