// Forward of the FP8 fake-quantised linear layer (Alg. 2 of the paper, with the scaled quantiser of App. B.2/B.3):
//     x_fp8 = E4M3(clamp(x / s_x, +-448)) * s_x   per token,          s_x = max(amax(x_i), 1e-8) / 448
//     W_fp8 = E4M3(clamp(W / s_W, +-448)) * s_W   per output channel, s_W likewise
//     y = x_fp8 W_fp8^T + b
// Two launches.  quantise_rows_kernel turns both bf16 matrices into E4M3 codes plus one fp32 scale per row; fp8_gemm_kernel
// multiplies the code matrices on v_mfma_f32_32x32x64_f8f6f4 (products of two E4M3 numbers are exact in the fp32
// accumulator) and applies s_x[i] s_W[o] and the bias in its epilogue.
//
// Between them the codes lie in fragment order, the order in which the matrix unit's operands are read: rows in groups
// of 32, of a group one 64-byte slice of K after the other, a slice as four runs of 16-byte pieces (piece (h,g) of row r:
// K bytes 32 g + 16 h .. + 15; runs ordered h, g; a run holds the group's rows one after the other).  A slice of a group is
// one operand of the MFMA and 2 KB of consecutive memory, so tiles reach LDS as plain 1 KB copies of consecutive bytes
// and leave it as 16-byte reads of consecutive lanes: no swizzle, no bank conflicts, whole lines, any K step.  The last
// group holds the rows that are there (R < 32: its runs are 16 R bytes), so the matrix takes rows x K bytes as before.
#include "sla_common.hpp"
#include "sla_kernels.hpp"

#include <type_traits>

namespace sla {

namespace {
constexpr int kSlice = 64;                           // bytes (= E4M3 elements) of K per slice: one MFMA
constexpr int kFrag = 32 * kSlice;                   // bytes of a slice of a full group
}  // namespace

// codes and scales of the rows of one matrix [rows, cols] (cols a multiple of 128), in fragment order
struct RowsIn {
    const uint16_t *X;
    long rows;
    uint8_t *codes;
    float *scales;
};

// A workgroup takes half a group, 16 rows: lane 4 r + c of wave w reads channels 64 s + 16 c .. + 15 of row r for the slices
// s = w, w + 4, ... (a quad reads one 128-byte line), holds them in registers through the maximum over the row (quad, then
// the four waves through LDS) and writes a piece of sixteen codes per slice: runs of 256 bytes.  Rows of more than 256 SL
// channels are read twice (ONE = false).  HBM bound (2 bytes in, 1 out per element) once the division is BlockDivisor's
// three instructions: with the division's own expansion the vector unit took as long as the memory.
// The first half groups belong to matrix a, the others to b: the few rows of the weights would be a launch of their own,
// most of which is waiting.  Measured: 43968 + 3072 rows of 1024 in 25 us = 5.5 TB/s (two launches, a row per wave read twice, with
// the division's expansion: 32 + 5.3 us); 1374 + 3072 rows 8.6 us (4.3 + 7.3 us and the gap between them).
template <int SL, bool ONE>                          // slices per wave and pass; rows of one pass
__global__ __launch_bounds__(256) void quantise_rows_kernel(RowsIn ma, RowsIn mb, int cols)
{
    asm volatile("" ::"s"(ma.X), "s"(ma.rows), "s"(ma.codes), "s"(ma.scales), "s"(mb.X), "s"(mb.rows), "s"(mb.codes), "s"(mb.scales), "s"(cols));      // all kernel arguments in one batch of scalar loads, here
    __shared__ float red[4][16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 3, r0 = lane >> 2;
    const long groups_a = (ma.rows + 31) / 32, blk = blockIdx.x >> 1;
    const bool first = blk < groups_a;
    const RowsIn m = first ? ma : mb;
    const long grp = first ? blk : blk - groups_a;
    const int R = (int)min(32L, m.rows - 32 * grp), row = 16 * (int)(blockIdx.x & 1) + r0;    // rows of the group (>= 1), this lane's
    const uint16_t *const x = m.X + (32 * grp + min(row, R - 1)) * cols + 16 * c;    // rows past the end repeat the last one
    const int slices = cols / kSlice, passes = ONE ? 1 : (slices + 4 * SL - 1) / (4 * SL);
    uint32_t w[SL][8];
    auto load = [&](int p) {
#pragma unroll
        for (int k = 0; k < SL; ++k) {               // and slices: no predicate, and the maximum is the same
            const uint16_t *const at = x + min((p * SL + k) * 4 + wave, slices - 1) * kSlice;
            const uint4 u = *(const uint4 *)at, v = *(const uint4 *)(at + 8);
            w[k][0] = u.x; w[k][1] = u.y; w[k][2] = u.z; w[k][3] = u.w;
            w[k][4] = v.x; w[k][5] = v.y; w[k][6] = v.z; w[k][7] = v.w;
        }
    };
    float amax = 0.f;
    for (int p = 0; p < passes; ++p) {
        load(p);
#pragma unroll
        for (int k = 0; k < SL; ++k)
#pragma unroll
            for (int q = 0; q < 8; ++q) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(w[k][q])), fabsf(bf16_hi(w[k][q]))));
    }
    amax = fmaxf(amax, __shfl_xor(amax, 1, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 2, 64));
    if (c == 0) red[wave][r0] = amax;
    __syncthreads();
    const float scale = fmaxf(fmaxf(fmaxf(red[0][r0], red[1][r0]), fmaxf(red[2][r0], red[3][r0])), 1e-8f) / 448.0f;
    if (wave == 0 && c == 0 && row < R) m.scales[32 * grp + row] = scale;
    uint8_t *const out = m.codes + 32 * grp * cols + (((c & 1) * 2 + (c >> 1)) * R + row) * 16;
    const BlockDivisor divide(scale);
    for (int p = 0; p < passes; ++p) {
        if (!ONE) load(p);
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            const int s = (p * SL + k) * 4 + wave;
            if (s < slices && row < R) *(uint4 *)(out + (size_t)s * R * kSlice) = quantise16(w[k], divide);
        }
    }
}

hipError_t launch_quantise_rows(const void *Xa, long rows_a, void *codes_a, float *scales_a, const void *Xb, long rows_b, void *codes_b,
                                float *scales_b, int cols, hipStream_t st)
{
    const RowsIn a = {(const uint16_t *)Xa, rows_a, (uint8_t *)codes_a, scales_a}, b = {(const uint16_t *)Xb, rows_b, (uint8_t *)codes_b, scales_b};
    const unsigned grid = (unsigned)(2 * ((rows_a + 31) / 32 + (rows_b + 31) / 32));
    if (cols <= 1024)      quantise_rows_kernel<4, true><<<grid, 256, 0, st>>>(a, b, cols);
    else if (cols <= 2048) quantise_rows_kernel<8, true><<<grid, 256, 0, st>>>(a, b, cols);
    else                   quantise_rows_kernel<8, false><<<grid, 256, 0, st>>>(a, b, cols);
    return hipGetLastError();
}

struct QkvOut {
    uint8_t *codes[3];          // Q, K, V codes, [B,N,H,64]
    float *scales[3];           // [B,H,ceil(N/blk)], blk = bq for Q, 64 for K and V
    int N, H, bq;
};

#ifdef SLA_PROBE_TIME   /* timing probe only: cycle counter of one wave at the phase boundaries of its tile */
__device__ unsigned long long sla_gemm_probe_times[16];
#define SLA_GT(pt) do { if (gprobe) { const unsigned long long t_ = __builtin_readcyclecounter(), r_ = __builtin_amdgcn_s_memrealtime(); if ((threadIdx.x & 63) == 0) { sla_gemm_probe_times[pt] = t_; sla_gemm_probe_times[8 + pt] = r_; } } } while (0)
#else
#define SLA_GT(pt)
#endif

// Y[i][o] = (sum_k A8[i][k] W8[o][k]) * sa[i] * sw[o] + bias[o];  A8 [M,K], W8 [O,K] E4M3 codes in fragment order, K a multiple of 128.
//
// Workgroup tile 64 TB tokens x 128 channels, four waves as 2 x 2, wave tile 32 TB tokens x 64 channels = TB x 2 MFMA tiles.
// The kernel forms D[o][i] (W as the A operand), so that four consecutive accumulator registers of a lane are four
// consecutive channels of one token.  K steps of one slice, three stages in LDS, copies two to three steps ahead of the
// products, one barrier per step (the schedule is written out at the loop).  TB = 4 holds 128 accumulators per wave and 75 KB
// of LDS: two workgroups share a CU, and the start and the epilogue of one (which take as long as its products) run under the
// products of the other.  Measured on 43968 x 1024 -> 3072: 143-150 us with the qkv epilogue (1.9 PFLOP/s), 165-170 us with bf16
// output, against 292 and 190 us of tiles of 256 x 256 at one workgroup per CU (sixteen fragment reads per thirty-two products,
// but a quarter of a tile's life start and epilogue with nothing beside them, half of it with the quantiser, and 2064 tiles in
// nine rounds of 256).  What bounds it now: the clock, which falls to 1.2-1.5 GHz under this load; the matrix unit is busy 54 %
// of the cycles (47 % with bf16 output), and a third of a tile's life is the quantiser's epilogue.
//
// QKV: the layer is the qkv projection in front of the attention (O = 3 H 64 output channels ordered [q|k|v][head][64])
// and the epilogue, instead of storing y, quantises it per (head, token block) with the scaled E4M3 quantiser of
// App. B.2 -- the form sla_forward takes E4M3 inputs in -- and stores codes [B,N,H,64] and scales [B,H,blocks] of Q, K
// and V directly.  A wave's 64 channels are one head and its tokens are whole token blocks (TB = 2: half of a 128-token
// block of Q, the other half being the neighbour wave's), so the bf16 values stay in the accumulator registers through the
// block's maximum, the division (BlockDivisor) and the conversion: the arithmetic of quantise_e4m3_kernel on the y that the
// unfused layer would store, hence the same bits.  Token blocks never straddle a tile (the host checks).
template <int TB, bool QKV>
__global__ __launch_bounds__(256, 2) void fp8_gemm_kernel(const uint8_t *__restrict__ A8, const float *__restrict__ sa,
                                                          const uint8_t *__restrict__ W8, const float *__restrict__ sw,
                                                          const uint16_t *__restrict__ bias, int M, int O, int K, int n_ot,
                                                          int total, uint16_t *__restrict__ Y, QkvOut qkv)
{
    asm volatile("" ::"s"(A8), "s"(sa), "s"(W8), "s"(sw), "s"(bias), "s"(M), "s"(O), "s"(K), "s"(n_ot), "s"(total), "s"(Y), "s"(qkv.codes[0]), "s"(qkv.codes[1]), "s"(qkv.codes[2]),
                 "s"(qkv.scales[0]), "s"(qkv.scales[1]), "s"(qkv.scales[2]), "s"(qkv.N), "s"(qkv.H), "s"(qkv.bq));      // all kernel arguments in one batch of scalar loads, here
    constexpr int kTok = 64 * TB;                                                // tokens per workgroup tile
    constexpr int kStage = (kTok + 128) * kSlice;                                // token groups, then the four channel groups
    __shared__ __attribute__((aligned(1024))) uint8_t smem[3 * kStage + (256 + kTok) * 4 + 16];
    float *const cs = (float *)(smem + 3 * kStage), *const ts = cs + 256, *const red = ts + kTok;    // channel scales, biases; token scales
    // channel tile fastest: the workgroups that share a token tile run side by side on one XCD, so the activations come
    // from HBM once; the weight matrix (a few MB) stays in every XCD's L2
    const int item = (int)xcd_remap(blockIdx.x, total);
    if (item >= total) return;
#ifdef SLA_PROBE_TIME
    const bool gprobe = __builtin_amdgcn_readfirstlane((int)(item == total / 2 + 5 && threadIdx.x < 64)) != 0;
#endif
    SLA_GT(0);
    const int it = (int)((unsigned)item / (unsigned)n_ot), ot = item - it * n_ot;
    const int i0 = it * kTok, o0 = ot * 128;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);                  // uniform: LDS destinations of the copies sit in scalar registers
    const int wo = (wave >> 1) * 64, wi = (wave & 1) * (32 * TB);                // wave's first channel / token within the tile

    // copies: a slice of a group is two copies of 1 KB (h = 0, 1: lane g * 32 + r brings piece (h,g) of row r; rows and
    // groups past the end repeat the last one: their results are never stored).  Wave w makes copies TB w .. TB w + TB - 1 of
    // the token tile's 4 TB and copies 2 w, 2 w + 1 of the channel tile's 8.
    constexpr int kGA = (TB + 1) / 2;                                            // token groups the wave copies from
    uint32_t va[TB], vw[2];
    int stride_a[kGA], stride_w;                                                 // bytes from one slice of a group to the next
    auto group = [](int rows, int first, int gl, int &R) {                       // group gl behind row `first`, clamped to the matrix
        const int grp = min(first / 32 + gl, (rows - 1) / 32);
        R = min(32, rows - 32 * grp);
        return grp;
    };
#pragma unroll
    for (int x = 0; x < TB; ++x) {
        const int id = wave * TB + x;
        int R;
        const int grp = group(M, i0, id >> 1, R);
        va[x] = (uint32_t)grp * 32u * (uint32_t)K + (uint32_t)((((id & 1) * 2 + g) * R + min(l32, R - 1)) * 16);
        stride_a[x >> 1] = R * kSlice;
    }
    {
        int R;
        const int grp = group(O, o0, wave, R);
#pragma unroll
        for (int x = 0; x < 2; ++x) vw[x] = (uint32_t)grp * 32u * (uint32_t)K + (uint32_t)(((x * 2 + g) * R + min(l32, R - 1)) * 16);
        stride_w = R * kSlice;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
    auto copy_one = [&](int k, uint32_t dst, int x) {                            // copy x of slice k of every group, into the stage at dst
        if (x < TB) copy_1k_to_lds(A8 + (size_t)((uint32_t)k * (uint32_t)stride_a[x >> 1]), va[x], dst + (wave * TB + x) * 1024);
        else        copy_1k_to_lds(W8 + (size_t)((uint32_t)k * (uint32_t)stride_w), vw[x - TB], dst + kTok * kSlice + (wave * 2 + x - TB) * 1024);
    };
    auto issue = [&](int k, uint32_t dst) {
#pragma unroll
        for (int x = 0; x < TB + 2; ++x) copy_one(k, dst, x);
    };
    const float sc = sw[min(o0 + (tid & 127), O - 1)];                           // scale and bias of channel o0 + tid % 128, scale of token i0 + tid
    const float bc = bias ? bf16_bits_to_f32(bias[min(o0 + (tid & 127), O - 1)]) : 0.f;
    const float sx = sa[min(i0 + tid, M - 1)];

    const int ksteps = K / kSlice;                                               // even, at least 2
    // Large launches: workgroups that share an operand tile run at the same time and would ask the same L2 channels for the
    // same lines at the same moment; each starts its K loop at a different step instead.  The sum over K is then taken in a
    // rotated order, which depends on the tile alone and is the same with and without the qkv epilogue.
    int k2 = TB == 4 ? 2 * (int)((unsigned)item % (unsigned)(ksteps / 2)) : 0;                       // slice that the next issue() copies
    auto advance = [&] { k2 = k2 + 1 == ksteps ? 0 : k2 + 1; };
    issue(k2, lds_base);
    advance();
    issue(k2, lds_base + kStage);
    advance();
    if (ksteps > 2) {
        issue(k2, lds_base + 2 * kStage);
        advance();
    }
    if (tid < 128) { cs[tid] = sc; cs[128 + tid] = bc; }                         // published by the barriers of the loop, read in the epilogue
    if (tid < kTok) ts[tid] = sx;

    f32x16 acc[2][TB];                                                          // [channel sub-tile][token sub-tile]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
    auto frag = [&](const uint8_t *slice) {                                      // operand of one MFMA: K bytes 32 g .. 32 g + 31 of row l32
        const uint4 u0 = *(const uint4 *)(slice + lane * 16), u1 = *(const uint4 *)(slice + 1024 + lane * 16);
        i32x8 f;
        f[0] = u0.x; f[1] = u0.y; f[2] = u0.z; f[3] = u0.w; f[4] = u1.x; f[5] = u1.y; f[6] = u1.z; f[7] = u1.w;
        return f;
    };
    // Step ks: its operands are in registers, all but those that the first half does not need for certain; first half of the
    // products (by token sub-tile); wait until the copies of step ks + 1 have landed (asked for two steps ago) and the own
    // reads have returned, barrier: stage (ks + 1) % 3 is whole, and stage ks % 3 has been read by everybody; second half of
    // the products, and between them the reads of step ks + 1 (a token operand is read again as soon as its products are
    // issued, the channel operands have two sets) and the copies of step ks + 3 into stage ks % 3.  A wave by itself so keeps
    // the matrix unit busy across the barrier, which matters while the other workgroup of the CU is in its epilogue.
    constexpr int kHalf = (TB + 1) / 2, kCopies = TB + 2;
    const uint8_t *const At = smem + (wave & 1) * TB * kFrag, *const Wt = smem + kTok * kSlice + (wave >> 1) * 2 * kFrag;
    i32x8 wf[2][2], af[TB];
    uint32_t stage = 0;                                                          // of the step whose products run
#define SLA_SB() __builtin_amdgcn_sched_barrier(0)
    auto mma = [&](int set, int b) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf[set][a], af[b], acc[a][b], 0, 0, 0, 0, 0, 0);
    };
    auto step = [&](auto set_, auto copy_, auto wait_, auto last_) {
        constexpr int set = decltype(set_)::value, wait = decltype(wait_)::value;
        constexpr bool copy = decltype(copy_)::value, last = decltype(last_)::value;
#pragma unroll
        for (int b = 0; b < kHalf; ++b) mma(set, b);
        SLA_SB();
        const uint32_t next = stage == 2 * kStage ? 0 : stage + kStage;
        if constexpr (!last) {
            if constexpr (wait == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopies) : "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);                                  // lgkmcnt(0) only, as a builtin: the compiler knows that the operands have arrived
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            SLA_SB();
#pragma unroll
            for (int a = 0; a < 2; ++a) wf[set ^ 1][a] = frag(Wt + next + a * kFrag);
#pragma unroll
            for (int b = 0; b < kHalf; ++b) af[b] = frag(At + next + b * kFrag);
            SLA_SB();
        }
        int done = 0;
#pragma unroll
        for (int b = kHalf; b < TB; ++b) {
            mma(set, b);
            SLA_SB();
            if constexpr (!last) af[b] = frag(At + next + b * kFrag);
            if constexpr (copy) {
#pragma unroll
                for (int x = 0; x < kCopies / 2; ++x)
                    if (b < TB - 1) copy_one(k2, lds_base + stage, done++);
            }
            SLA_SB();
        }
        if constexpr (copy) {
#pragma unroll
            for (int x = 0; x < kCopies; ++x)
                if (x >= done) copy_one(k2, lds_base + stage, x);
            advance();
        }
        stage = next;
    };
    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, 1>;
    using Yes = std::true_type;
    using No = std::false_type;
    if (ksteps > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kCopies) : "memory");
    else            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopies) : "memory");
    lds_barrier();
    SLA_GT(1);
#pragma unroll
    for (int a = 0; a < 2; ++a) wf[0][a] = frag(Wt + a * kFrag);
#pragma unroll
    for (int b = 0; b < TB; ++b) af[b] = frag(At + b * kFrag);
    if (ksteps > 2) {
        for (int ks = 0; ks < ksteps - 4; ks += 2) {
            step(Set0{}, Yes{}, Set1{}, No{});
            step(Set1{}, Yes{}, Set1{}, No{});
        }
        step(Set0{}, Yes{}, Set1{}, No{});
        step(Set1{}, No{}, Set1{}, No{});
    }
    step(Set0{}, No{}, Set0{}, No{});
    step(Set1{}, No{}, Set0{}, Yes{});
#undef SLA_SB
    SLA_GT(2);

    // Accumulator (a,b) register 4q+r of lane (l32, g): channel o0 + wo + 32a + 8q + 4g + r, token i0 + wi + 32b + l32.
    // y = acc * (s_token * s_channel) + bias, two roundings before the bf16 one (the scales first: acc times one of them alone can
    // overflow where y does not).  No staging in LDS: lanes l and l + 32 hold
    // the other half of each other's channels, and v_permlane32_swap brings the pieces of a 16-byte store together.
    float4 sw4[2][4], bi4[2][4];
    float si[TB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = wo + 32 * a + 8 * q + 4 * g;
            sw4[a][q] = *(const float4 *)(cs + c);
            bi4[a][q] = *(const float4 *)(cs + 128 + c);
        }
#pragma unroll
    for (int b = 0; b < TB; ++b) si[b] = ts[wi + 32 * b + l32];
    auto value = [&](int a, int b, int q, float (&v)[4]) {
        v[0] = fmaf(acc[a][b][4 * q + 0], si[b] * sw4[a][q].x, bi4[a][q].x);
        v[1] = fmaf(acc[a][b][4 * q + 1], si[b] * sw4[a][q].y, bi4[a][q].y);
        v[2] = fmaf(acc[a][b][4 * q + 2], si[b] * sw4[a][q].z, bi4[a][q].z);
        v[3] = fmaf(acc[a][b][4 * q + 3], si[b] * sw4[a][q].w, bi4[a][q].w);
    };
    auto swap32 = [](uint32_t &lo, uint32_t &hi) {                               // upper lanes of lo <-> lower lanes of hi
        const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        lo = r[0];
        hi = r[1];
    };
    if constexpr (!QKV) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int i = i0 + wi + 32 * b + l32;
            uint16_t *const y = Y + (size_t)i * O;
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int q = 0; q < 4; q += 2) {
                    float v0[4], v1[4];
                    value(a, b, q, v0);
                    value(a, b, q + 1, v1);
                    uint32_t x0 = pack_bf16(v0[0], v0[1]), y0 = pack_bf16(v0[2], v0[3]), x1 = pack_bf16(v1[0], v1[1]), y1 = pack_bf16(v1[2], v1[3]);
                    swap32(x0, x1);                                              // lower lanes: channels 8q .. 8q+7, upper: 8q+8 .. 8q+15
                    swap32(y0, y1);
                    const int o = o0 + wo + 32 * a + 8 * q + 8 * g;
                    if (i < M && o < O) *(uint4 *)(y + o) = make_uint4(x0, y0, x1, y1);      // O is a multiple of 8: a piece is in or out as a whole
                }
        }
    } else {
        const int N = qkv.N, H = qkv.H, ch0 = o0 + wo, t0 = i0 + wi;              // the wave's head and its first token
        const bool in = ch0 < O && t0 < M;
        const int which = ch0 / (H * 64), h = (ch0 - which * H * 64) >> 6;
        const int blk = which == 0 ? qkv.bq : kBK;
        constexpr int kBlocks = TB / 2;                                          // 64-token blocks of the wave's tile
        float amax[kBlocks];
#pragma unroll
        for (int t = 0; t < kBlocks; ++t) amax[t] = 0.f;
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            float m = 0.f;
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
                    value(a, b, q, v);
#pragma unroll
                    for (int r = 0; r < 4; r += 2) {                             // from here on the register holds y, rounded to bf16
                        const uint32_t p = pack_bf16(v[r], v[r + 1]);
                        acc[a][b][4 * q + r] = bf16_lo(p);
                        acc[a][b][4 * q + r + 1] = bf16_hi(p);
                        m = max3_abs(m, bf16_lo(p), bf16_hi(p));
                    }
                }
            if (t0 + 32 * b + l32 < M) amax[b >> 1] = fmaxf(amax[b >> 1], m);     // rows past the end are not part of the block
        }
#pragma unroll
        for (int t = 0; t < kBlocks; ++t) amax[t] = wave_max_dpp(amax[t]);
        if constexpr (TB == 2) {
            if (lane == 0) red[wave] = amax[0];
            lds_barrier();
            if (blk == 128) amax[0] = fmaxf(amax[0], red[wave ^ 1]);
        } else if (blk == 128) amax[0] = amax[1] = fmaxf(amax[0], amax[1]);
        if (!in) return;                                                         // uniform over the wave, no barrier below
        const int nblk_seq = (N + blk - 1) / blk, bt = t0 / N, tin = t0 - bt * N;
        uint8_t *const codes = qkv.codes[which] + ((size_t)t0 * H + h) * 64 + 16 * g;
        float *const scales = qkv.scales[which] + ((size_t)bt * H + h) * nblk_seq;
#pragma unroll
        for (int t = 0; t < kBlocks; ++t) {
            if (t0 + 64 * t >= M) break;                                         // uniform over the wave
            const float scale = fmaxf(amax[t], 1e-8f) / 448.0f;
            if (lane == 0 && (tin + 64 * t) % blk == 0) scales[(tin + 64 * t) / blk] = scale;
            const BlockDivisor divide(scale);
#pragma unroll
            for (int b = 2 * t; b < 2 * t + 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    uint32_t d[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float y[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) y[r] = fminf(fmaxf(divide(acc[a][b][4 * q + r]), -448.0f), 448.0f);
                        d[q] = pack_e4m3(y[0], y[1], y[2], y[3]);
                    }
                    swap32(d[0], d[2]);                                          // lower lanes: channels 0 .. 15 of the sub-tile, upper: 16 .. 31
                    swap32(d[1], d[3]);
                    if (t0 + 32 * b + l32 < M) *(uint4 *)(codes + (size_t)(32 * b + l32) * H * 64 + 32 * a) = make_uint4(d[0], d[2], d[1], d[3]);
                }
        }
    }
#ifdef SLA_PROBE_TIME
    SLA_GT(3);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    SLA_GT(4);
#endif
}
#ifdef SLA_PROBE_TIME
extern "C" int sla_probe_read_gemm(unsigned long long *dst) { return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(sla_gemm_probe_times), sizeof(unsigned long long) * 16); }
#endif

// 256-token tiles where the launch has 512 of them, one per slot of the chip (two workgroups per CU)
static bool lin_wide_tiles(int M, int O) { return (long)((M + 255) / 256) * ((O + 127) / 128) >= 512; }

namespace {
template <int TB, bool QKV>
hipError_t launch_gemm(const void *A8, const float *sa, const void *W8, const float *sw, const void *bias, int M, int O, int K, void *Y,
                       const QkvOut &q, hipStream_t st)
{
    const int n_it = (M + 64 * TB - 1) / (64 * TB);
    const int n_ot = (O + 127) / 128;
    const long total = (long)n_it * n_ot;
    if (total > 0x7FFFFFF0L) return hipErrorInvalidValue;
    fp8_gemm_kernel<TB, QKV><<<(unsigned)xcd_grid(total), 256, 0, st>>>((const uint8_t *)A8, sa, (const uint8_t *)W8, sw, (const uint16_t *)bias, M, O, K,
                                                                        n_ot, (int)total, (uint16_t *)Y, q);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_fp8_gemm(const void *A8, const float *sa, const void *W8, const float *sw, const void *bias, int M, int O, int K,
                           void *Y, hipStream_t st)
{
    // 128-token tiles from 400 of them on: 420 tiles (2600 x 1920 -> 2496) take 27.5 us, their halves 31.8; 448 (3500 x 2048 ->
    // 2048) 30.5 against 33.8; 384 (2000 x 1024 -> 3072) the same; 264 (1374 x 1024 -> 3072) 19.3 against 18.8
    if (lin_wide_tiles(M, O)) return launch_gemm<4, false>(A8, sa, W8, sw, bias, M, O, K, Y, QkvOut{}, st);
    if ((long)((M + 127) / 128) * ((O + 127) / 128) >= 400) return launch_gemm<2, false>(A8, sa, W8, sw, bias, M, O, K, Y, QkvOut{}, st);
    return launch_gemm<1, false>(A8, sa, W8, sw, bias, M, O, K, Y, QkvOut{}, st);
}

int fp8_gemm_qkv_token_tile(int M, int H) { return lin_wide_tiles(M, 3 * H * 64) ? 256 : 128; }

hipError_t launch_fp8_gemm_qkv(const void *A8, const float *sa, const void *W8, const float *sw, const void *bias, int B, int N, int H, int K,
                               int bq, void *const codes[3], float *const scales[3], hipStream_t st)
{
    const int M = B * N, O = 3 * H * 64;
    QkvOut q;
    for (int w = 0; w < 3; ++w) { q.codes[w] = (uint8_t *)codes[w]; q.scales[w] = scales[w]; }
    q.N = N; q.H = H; q.bq = bq;
    if (lin_wide_tiles(M, O)) return launch_gemm<4, true>(A8, sa, W8, sw, bias, M, O, K, nullptr, q, st);
    return launch_gemm<2, true>(A8, sa, W8, sw, bias, M, O, K, nullptr, q, st);
}

}  // namespace sla
