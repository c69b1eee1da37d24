// Block-sparse flash attention over the critical key blocks of each query block, fused with
// the linear-branch output, the projection and the sum (Alg. 1 steps 4-5, 9, 10; eq. (1)):
//     O_i = softmax_{t' in critical blocks}(Q_i K_t'^T * scale) V_t'
//           + [ phi(Q_i) H_i / (phi(Q_i) . Z_i) ] W_proj
//
// Everything is kept transposed so that a lane owns query rows:
//     S^T[t'][q]  = K (A operand, LDS rows)   x  Q^T (B operand, registers)
//     O^T[e][q]  += V^T (A operand, LDS)      x  P^T (B operand = the S^T accumulators, re-used in place: no LDS round trip)
// With the 32x32x16 MFMA a lane holds column q = lane%32 of the 32x32 result, rows 8a + 4g + b (g = lane/32; register 4a+b).
// The B operand of the second product takes accumulator registers 8u..8u+7, i.e. keys 16s + 8a' + 4g + b; the V^T rows are read
// with exactly that key permutation: the states kernel leaves V^T of every key block in that order, so a V^T fragment is one
// 16-byte LDS read like a K fragment.
//
// Work decomposition.  One workgroup per (b, h, query block).  A wave owns 64 query rows in two groups (A, B) of 32 and takes 32
// keys at a time (a unit is 32 keys x 32 rows).  RH: halves of 64 rows in a query block, KS: parts into which the keys of every key
// block are split, one wave for each combination.  128-row blocks run as RH = 2, KS = 1 and, in launches too small to fill the chip
// that way, as RH = 2, KS = 2; 64-row blocks as RH = 1, KS = 2.  With KS = 2 the two waves that share rows exchange a group each
// at the end (accumulators, reference exponent and row sums through LDS) and finish 32 rows each.
// Why 64 rows per wave: every K and V^T fragment read from LDS feeds the products of both groups.  With 32 rows per wave (the form
// before) the fragment reads took two thirds of the LDS bandwidth.  The two groups are also what the software pipeline needs: while
// the vector unit runs the softmax of one group's unit, the matrix unit runs S^T of the other group's next unit and O += V P of its
// last one; no second S^T buffer is held, and the 64 rows fit 256 registers: two waves per SIMD, four workgroups of two waves
// per CU.
//
// Steps.  Units s = 0, 1, ... of a wave (KS = 1: tile s / 2, half s % 2; KS = 2: tile s, the wave's half of it); two steps for each:
//   step A(s): softmax of A's unit s    beside  row sums of B's last weights, S_B(s) = K(s) Q_B (then K(s+1) is read), O_B += V(s-1) P_B(s-1)
//   step B(s): softmax of B's unit s    beside  row sums of A's weights, S_A(s+1) = K(s+1) Q_A, O_A += V(s) P_A(s)
// V(s) is read from LDS during step A(s) into the other of two fragment buffers.
//
// Arithmetic of the weights.  P is rounded to fp16 (11 significant bits) and V^T arrives as fp16 from the states
// kernel (bf16 or E4M3 values are exact in fp16 once divided by the power of two the states kernel picks per key
// block; its base-2 logarithm comes in `lvs` and is added to the exponent of the weights, so the product is
// unchanged).  The second product runs on the fp16 MFMA at the rate of the bf16 one with an eighth of the rounding
// error on the weights.  That margin pays for a reference exponent that is raised only when weights come to lie well above it:
// the accumulators are rescaled a few times per row instead of once per tile, and the softmax of a unit needs nothing from
// other lanes before its exponentials.  Whether the reference has to be raised shows in the unit's row sums (formed on the matrix
// unit from the fp16 weights), two instructions a unit; then the unit is repaired (see there).  A maximum over the exponents in front of
// the exponentials, the form before, takes ten of the unit's 52 vector instructions, and vector issue is what bounds the loop.
// A repair reads its keys again from global memory, some 4000 cycles with the wait of the other waves, so the tiles behind one are
// prescanned (see there): where a logit has left the range another is likely to, and a prescan costs some 1350 a tile, raise included.
// Tiles whose V scale is far from the list's are prescanned too, for their row sums.  Forward on given labels with 16 heads, against a repair
// for every unit that passes 2^8 or is of such a tile: 43968 tokens, V of every second block 2^-10 of the others' 1270 -> 805 us; one
// block in sixteen 752 -> 617; keys four times as long 674 -> 601, ten times 854 -> 676, growing along the sequence by twenty 1264 -> 720;
// 60000 tokens in E4M3, the same five: 1622 -> 966, 968 -> 779, 830 -> 732, 1057 -> 800, 1587 -> 864; 10992 tokens in 64-row blocks 145 -> 108,
// 112 -> 95, 113 -> 95, 134 -> 102, 140 -> 103.  (With a maximum in front of every unit instead, the form before: 43968 tokens 874, 661, 630,
// 631, 684; E4M3 1226, 898, 771, 794, 878; 10992 tokens 112, 104, 89, 90, 93.)  Benign keys: 546 -> 549, 704 -> 699, 92 -> 90.
//
// Memory pipeline.  K and V^T tiles go from global memory straight into LDS (buffer loads, no staging registers).  K has four
// slots of half a tile, V^T two of a tile: 33 KB, so that four workgroups fit a CU.  Iteration c (tile c) reads V^T tile c and, KS = 1,
// K slices 2c+1 and 2c+2, KS = 2, K tile c+1; they were asked for an iteration earlier (behind its first step), landed at its
// barrier, and the barrier frees the slots of what was read before.  Rows are stored unpadded with the 16-byte chunk
// index XOR-ed by row bits (applied on the global side of the copy), which keeps the fragment reads free of bank conflicts.  The
// copies are inline assembly, invisible to the compiler's wait-count insertion (which would drain them before every LDS
// read), and are awaited by explicit s_waitcnt vmcnt(0).
//
// E4M3 inputs.  S^T is one v_mfma_f32_32x32x64_f8f6f4 per 32 keys (the whole head dimension is the K dimension of
// the instruction; products of two E4M3 numbers are exact in the fp32 accumulator), with the per-block scales
// folded into the exp2 constant.  P is NOT cast to E4M3: three mantissa bits on the softmax weights put the output
// error at several percent of its RMS, above the 6e-2 bar; the second product is the fp16 one described above, with
// the V block scale in the exponent of the weights.
//
// Epilogue (per 32 rows, all MFMA): O_lin^T = Hq^T-tile x phi(Q)^T, scaled by 1/(phi(Q).Z),
// then W^T x O_lin^T, added to the normalised sparse output and stored as bf16.
//
// What bounds it: the issue of vector instructions beside the MFMA (42 and 10 per unit), LDS reads and tile copies, each about a tenth
// of the time (left out one at a time), prologue and epilogue (a sixth on lists of 34, over 40 % on lists of 9).  Against 32 rows per wave
// with a maximum over the exponents and a separate careful form of a step, launches of 16 heads: 43968 tokens, lists of 34, bf16 497 ->
// 420 us; 137400 tokens, lists of 64, e4m3 2300 -> 1960; 17856 tokens, lists of 14, bf16 106 -> 96; 10992 tokens in 64-row blocks, lists
// of 9, 58.5 -> 55.5.  Of that, 64 rows per wave and buffer copies (a third of the scalar instructions) gave 9 %, the check on the row
// sums and the order of the products 5 %.
#include "attend_common.hpp"
#include "sla_kernels.hpp"

#include <type_traits>

namespace sla {

// A unit whose weights (V scale included) add up to more than this has the reference raised to its exact maximum.  fp16 holds weights
// below 2^16.  The closer the largest weights are to the reference, the more often the largest one is 1 exactly, and the smaller the error: with
// 2^8 it is the same on the benchmark's keys, 14 % less on keys three times as long (1.03e-4 against 0.88e-4 of the result, 1.04e-4 with
// an exact maximum wherever a weight passes 2^12), but such keys then repair often (43968 tokens, keys four times as long: 709 us against 601).
constexpr float kRepair = 32768.0f;
// A prescan raises the reference of rows with weights above 2^kAhead: 32 of those are within kRepair.
constexpr float kAhead = 10.0f;
// Tiles that are prescanned behind a repair, or a prescan that raised.  (Four: 627 us instead of 601 on the keys above, no difference on others.)
constexpr int kHot = 2;
// A row is spoilt (see repair) if its largest exponent lies this far above its own maximum.
constexpr float kSpoilt = 12.0f;
// A key block whose V scale differs from the list's reference by more than 2^kTinyV either way, or is as far below the largest one
// of the list so far: the factor that divides the scale out of the row sums again would leave the range of fp16, so they are formed
// in fp32 (prescan).
constexpr float kTinyV = 8.0f;

#ifdef SLA_PROBE_TIME   /* timing probe only: cycle counter of one wave at five points of every tile */
__device__ unsigned long long sla_wg_times[2 * 32768];      // 100 MHz clock at the start and the end of every workgroup (the first 32768)
__device__ unsigned long long sla_probe_times[64 * 8];
#define SLA_TP(row, pt) do { if (probe_on) { const unsigned long long t_ = __builtin_readcyclecounter(); if (lane == 0) tprobe[(row) * 8 + (pt)] = t_; } } while (0)
#define SLA_T(c, pt) do { if ((c) < 61) SLA_TP(c, pt); } while (0)      /* rows 61..63: epilogue, prologue, wave life */
#else
#define SLA_TP(row, pt)
#define SLA_T(c, pt)
#endif

// RH row halves of 64 rows times KS parts of the keys: one wave each
template <bool FP8, int RH, int KS>
struct AttendTile {
    static constexpr int KROWB = FP8 ? 64 : 128;                // bytes of a K row in LDS
    static constexpr int KSLICE = 32 * KROWB;                   // half a K tile
    static constexpr int VBYTES = 64 * 128;                     // V^T tile (fp16)
    static constexpr int VRING = 4 * KSLICE;                    // the V^T ring follows the K ring
    static constexpr int ZOFF = VRING + 2 * VBYTES;             // the Z row of the epilogue
    static constexpr int WOFF = ZOFF + 1024;                    // E4M3: W^T (bf16: in the K ring)
    static constexpr int WAVES = RH * KS;
    static constexpr int XOFF = WOFF + (FP8 ? 8192 : 0);        // KS = 2: reference exponents and row sums that the waves exchange, and, RH = 2,
    static constexpr int OOFF = XOFF + 512 * WAVES;             // the accumulators (RH = 1: in the rings)
    static constexpr int LDS = KS == 1 ? XOFF : RH == 1 ? OOFF : OOFF + 8192 * WAVES;
};

template <bool FP8, int RH, int KS>
__global__ __launch_bounds__(64 * RH * KS, 2) void attend_kernel(
    const void *__restrict__ Qp, const void *__restrict__ Kp, const uint16_t *__restrict__ Vp, const float *__restrict__ lvs,
    const float *__restrict__ sQ, const float *__restrict__ sK, RowMap rm,
    const int32_t *__restrict__ crit_idx, int k_c, const uint16_t *__restrict__ Hq, const uint16_t *__restrict__ WT,
    int proj_per_head, int phi, int H, int N, int Nqb, int Nkb, long total, float c_exp, uint16_t *__restrict__ O, float *__restrict__ O32)
{
    using T = AttendTile<FP8, RH, KS>;
    constexpr int ES = FP8 ? 1 : 2;                     // bytes per input element
    constexpr int A = 0, B = 1;                         // the two groups
    constexpr uint32_t kNaN2 = 0x7E007E00u;             // two fp16 NaN
    __shared__ __attribute__((aligned(1024))) uint8_t lds[T::LDS];
    // all kernel arguments in one batch of scalar loads (left to the compiler: a round trip in front of each first use)
    asm volatile("" ::"s"(Qp), "s"(Kp), "s"(Vp), "s"(lvs), "s"(sQ), "s"(sK), "s"(rm.bs), "s"(rm.hs), "s"(rm.ts), "s"(rm.H), "s"(crit_idx),
                 "s"(k_c), "s"(Hq), "s"(WT), "s"(proj_per_head), "s"(phi), "s"(H), "s"(N), "s"(Nqb), "s"(Nkb), "s"(total), "s"(c_exp), "s"(O), "s"(O32));
    const long work = xcd_remap(blockIdx.x, total);
    if (work >= total) return;                          // the whole workgroup leaves together
    const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#ifdef SLA_PROBE_TIME
    __shared__ unsigned long long tprobe[64 * 8];
    const bool probe_on = __builtin_amdgcn_readfirstlane((int)(work == total / 2 + 3 && wave_u == 1)) != 0;
    const unsigned long long tp_c0 = __builtin_readcyclecounter(), tp_r0 = __builtin_amdgcn_s_memrealtime();
    if (threadIdx.x == 0 && work < 32768) sla_wg_times[2 * work] = tp_r0;
#endif
    const long bh = (long)((unsigned)work / (unsigned)Nqb);      // (the grid fits 32 bits)
    const int i = (int)(work - bh * Nqb);
    const int kh = KS == 2 ? wave_u & 1 : 0;            // KS = 2: this wave's half of every tile
    // first row of this wave; group r has rows q0w + 32 (r ^ kh) ..: a wave finishes its group A and gives B away
    const int q0w = 64 * (RH * i + wave_u / KS);
    const size_t head = rm.head(bh);
    const int krowb = rm.ts * ES;                       // bytes between consecutive K rows
    const uint8_t *Kh = (const uint8_t *)Kp + head * ES;
    const uint8_t *Vh = (const uint8_t *)(Vp + (size_t)bh * Nkb * kBK * kD);
    const float *lvh = lvs + bh * Nkb;

    SLA_TP(62, 0);
    // the critical list first of all: everything in the prologue waits for it
    const int32_t *ci = crit_idx + work * (long)k_c;
    const int j0_first = lane < k_c ? ci[lane] : -1;
    // Q as the B operand of S^T: bf16 -> 4 K-steps of 8 channels (16s + 8g ..), e4m3 -> 32 channels (32g ..); loaded in the prologue
    bf16x8 qf[2][4];
    i32x8 q8[2];
    const float qscale = FP8 ? sQ[work] : 1.0f;         // scale blocks of Q are the query blocks

    // per-lane LDS byte offsets of the fragments (swizzled 16-byte chunks): koff[s] in a K slice, row l32, channel chunk of step s;
    // voff[ss] in a V^T tile, row l32 (+32 for channels 32..63), key chunk 2 ss + g; the tile's second half flips bit 6
    int koff[FP8 ? 2 : 4], voff[2];
#pragma unroll
    for (int s = 0; s < (FP8 ? 2 : 4); ++s)
        koff[s] = kh * T::KSLICE + (FP8 ? l32 * 64 + (((2 * g + s) ^ swz4(l32)) << 4) : l32 * 128 + (((2 * s + g) ^ swz8(l32)) << 4));
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) voff[ss] = l32 * 128 + (((4 * kh + 2 * ss + g) ^ swz8(l32)) << 4);

    f32x16 zero16;
#pragma unroll
    for (int x = 0; x < 16; ++x) zero16[x] = 0.f;
    f32x16 oacc[2][2] = {{zero16, zero16}, {zero16, zero16}};
    // Running state of the lane's two rows: reference exponent, row sums of the steps (formed on the matrix unit from the fp16 weights,
    // with 2^-scale as A operand where a row and a chunk of K belong together) and of the units repair() made again or prescan() summed.
    // For bf16 V that factor is a power of two; an E4M3 block's is not, and its rounding to fp16 would be an error of up to 2^-12 on all the
    // block's weights in the row sum.  So what fp16 leaves of it is the operand of a second row: register 0 has the sum, 1 the correction.
    float m_run[2] = {-3.4028235e38f, -3.4028235e38f}, l_full[2] = {0.f, 0.f};
    f32x4 lsum[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    float l_old[2][2] = {{0.f, 0.f}, {0.f, 0.f}};       // the two without the last unit
    // which half of TileInfo::inv2 this lane's operand repeats (a v_perm selector; 12: a zero byte)
    const uint32_t ones_sel = (((lane >> 2) ^ (lane >> 4)) & 1) || (lane & 2) ? 0x0c0c0c0cu : (lane & 1) ? 0x03020302u : 0x01000100u;
    f16x8 ones;

    // ragged block: only the last key block of the sequence can be short
    const int tail_rows = N & (kBK - 1), ragged_j = tail_rows ? Nkb - 1 : -1;
    // the list: a window of 64 entries in lanes
    int wbase = 0, d_j = 0;
    // (log2 of its V scale, exp2 constant, what divides the V scale out of the row sums)
    float d_lv = 0.f, d_cj = 0.f, lv_ref = 0.f, lv_top = -INFINITY;
    uint32_t d_inv2 = 0u;
    unsigned long long d_far = 0;                       // entries whose V scale is far from the reference
    float d_lim = 0.f;                                  // kRepair in units of the row sums
    int k = 0;                                          // leading valid entries
    {
        const int j0 = j0_first;
        unsigned long long ok = __ballot(j0 >= 0 && j0 < Nkb);
        d_j = (j0 >= 0 && j0 < Nkb) ? j0 : 0;
        if (ok != ~0ull) k = __builtin_ctzll(~ok);
        else {
            k = 64;
            for (int base = 64; base < k_c; base += 64) {
                const int idx = base + lane;
                const int j = idx < k_c ? ci[idx] : -1;
                ok = __ballot(j >= 0 && j < Nkb);
                if (ok == ~0ull) { k += 64; continue; }
                k += __builtin_ctzll(~ok);
                break;
            }
        }
        k = __builtin_amdgcn_readfirstlane(k);
    }
    // lv: scale of the lane's block; cj: exp2 constant of its tile
    auto window_scales = [&](bool first, float lv, float cj) __attribute__((always_inline)) {
        d_cj = cj;
        d_lv = relative_scale(lv, wbase + lane < k, first, lv_ref);
        lv_top = fmaxf(lv_top, wave_max_dpp(wbase + lane < k ? d_lv : -INFINITY));
        const bool far = !(fabsf(d_lv) <= kTinyV) || d_lv < lv_top - kTinyV;
        const float r = fast_exp2(-d_lv);
        // in fp16 and what that leaves; NaN for a ragged tile, which makes the row sums of its units NaN and sends them to repair; 0 for a V
        // scale far from the others': prescan forms the row sums
        d_inv2 = d_j == ragged_j ? kNaN2 : far ? 0u : pack_f16(r, FP8 ? r - (float)(_Float16)r : 0.f);
        d_far = __ballot(d_inv2 == 0u);
        d_lim = kRepair * r;
    };
    // softmax scale * log2(e) (* Q and K block scales for e4m3)
    auto exp_constant = [&](float sk) __attribute__((always_inline)) { return FP8 ? fmaxf(c_exp * qscale * sk, 1e-30f) : c_exp; };
    auto load_window = [&](int wb) __attribute__((always_inline)) {
        d_j = ci[min(wb + lane, k - 1)];                    // (entries behind the list repeat the last one)
        asm volatile("" : "+v"(d_j));
        wbase = wb;
        float lv = lvh[d_j], cj = exp_constant(FP8 ? sK[bh * Nkb + d_j] : 0.f);
        asm volatile("" : "+v"(lv), "+v"(cj));              // the loads complete here, not at some later first use
        window_scales(false, lv, cj);
    };
    auto entry_j = [&](int c) { return __builtin_amdgcn_readlane(d_j, c - wbase); };

    SLA_TP(62, 1);
    // ---- copies.  A K slice is four instructions of 8 rows (bf16) or two of 16 (e4m3), a V^T tile eight of 8; each wave issues
    // half of them.  The swizzle of a row group advances by 4 mod 8 from one 8-row instruction to the next: a flip of
    // offset bit 6 for odd ones (rows of 128 bytes), none for 64-byte rows.  They are buffer loads: the descriptor carries the tile's
    // address and, for the ragged block, the end of its last row, behind which zeros are read (masked later); the immediate offset
    // moves both the source and the LDS address, so a V^T tile takes one write of M0.
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_p)lds;
    const uint32_t ktile_bytes = (uint32_t)kBK * (uint32_t)krowb;
    const uint32_t lds_k = lds_base + wave_u * (T::KSLICE / 2), lds_v = lds_base + T::VRING + wave_u * (8192 / T::WAVES);
    const uint32_t half_bytes = 32u * (uint32_t)krowb;
    uint32_t vo_k[FP8 ? 1 : 2], vo_v[2];                // per-lane source offsets: K by instruction, V^T even and odd instructions
    {
        const uint32_t lr = FP8 ? lane >> 2 : lane >> 3;
        const uint32_t chunk = FP8 ? (uint32_t)((lane & 3) ^ swz4(lr)) << 4 : (uint32_t)((lane & 7) ^ swz8(lr)) << 4;
#pragma unroll
        for (int x = 0; x < (FP8 ? 1 : 2); ++x) vo_k[x] = (16 * wave_u + 8 * x + lr) * (uint32_t)krowb + (chunk ^ (x ? 64u : 0u)) - 1024u * x;      // (- the immediate offset)
        vo_v[0] = wave_u * (8192 / T::WAVES) + (lane >> 3) * 128 + ((uint32_t)((lane & 7) ^ swz8(lane >> 3)) << 4);
        vo_v[1] = vo_v[0] ^ 64u;
    }
    auto descriptor = [](const uint8_t *base, uint32_t records) __attribute__((always_inline)) {
        const uint64_t a = (uint64_t)base;
        return i32x4{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)records, 0x00027000};
    };
    // half h of the K tile of key block j (four waves: h = 0 is the whole tile); bytes up to the end of the last row there is, in a ragged block
    auto k_descriptor = [&](uint32_t j, int h) __attribute__((always_inline)) {
        const int rows = tail_rows - 32 * h;
        const uint32_t tail = rows > 0 ? (uint32_t)(rows - 1) * (uint32_t)krowb + T::KROWB : 0u;
        return descriptor(Kh + (uint64_t)j * ktile_bytes + (h ? half_bytes : 0u), (int)j == ragged_j ? tail : ~0u);
    };
    auto v_descriptor = [&](uint32_t j) __attribute__((always_inline)) { return descriptor(Vh + (uint64_t)j * (uint32_t)(kBK * kD * 2), ~0u); };
    // the half tile (four waves: the tile) kd describes into K slot `slot`
    auto request_K = [&](const i32x4 &kd, int slot) __attribute__((always_inline)) {
        uint32_t m0;
        if constexpr (FP8)
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds\n\ts_mov_b32 m0, %0"
                         : "=&s"(m0) : "v"(vo_k[0]), "s"(kd), "s"(lds_k + slot) : "memory");
        else
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                         "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds\n\ts_mov_b32 m0, %0"
                         : "=&s"(m0) : "v"(vo_k[0]), "v"(vo_k[FP8 ? 0 : 1]), "s"(kd), "s"(lds_k + slot) : "memory");
    };
    // a V^T tile (or any contiguous 8 KB) to LDS address dst (which includes this wave's half)
    auto request_tile = [&](const i32x4 &vd, uint32_t dst) __attribute__((always_inline)) {
        uint32_t m0;
        if constexpr (T::WAVES == 4)
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                         "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds\n\ts_mov_b32 m0, %0"
                         : "=&s"(m0) : "v"(vo_v[0]), "v"(vo_v[1]), "s"(vd), "s"(dst) : "memory");
        else
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                         "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds\n\tbuffer_load_dwordx4 %1, %3, 0 offen offset:2048 lds\n\t"
                         "buffer_load_dwordx4 %2, %3, 0 offen offset:3072 lds\n\ts_mov_b32 m0, %0"
                         : "=&s"(m0) : "v"(vo_v[0]), "v"(vo_v[1]), "s"(vd), "s"(dst) : "memory");
    };
    // The operands of the epilogue travel during the last tile (phase P): Hq^T into the V^T slot that is free, W^T into the two
    // K slots next to each other that are (slice 2c+1 is in the other pair), Z behind the rings.
    const uint8_t *Hi8 = Hq ? (const uint8_t *)(Hq + (size_t)work * kStateElems) : nullptr;
    const uint8_t *Wh8 = (const uint8_t *)(WT + (proj_per_head ? (size_t)((unsigned)bh % (unsigned)H) * kD * kD : 0));
    auto hq_off = [](int P) { return (uint32_t)(T::VRING + (P ^ 1) * T::VBYTES); };
    auto wt_off = [](int P) { return (uint32_t)(FP8 ? T::WOFF : (P ? 0 : 2 * T::KSLICE)); };
    auto request_epilogue = [&](int P) __attribute__((always_inline)) {
        if (Hq == nullptr) return;
        request_tile(descriptor(Hi8, ~0u), lds_base + hq_off(P) + wave_u * (8192 / T::WAVES));
        request_tile(descriptor(Wh8, ~0u), lds_base + wt_off(P) + wave_u * (8192 / T::WAVES));
        if (wave_u == 0) {                                  // 128 bytes, zeros behind them
            uint32_t m0;
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds\n\ts_mov_b32 m0, %0"
                         : "=&s"(m0) : "v"(lane_now() * 16), "s"(descriptor(Hi8 + 64 * kD * 2, 128)), "s"(lds_base + T::ZOFF) : "memory");
        }
    };

    // ---- per-tile constants (wave-uniform)
    struct TileInfo { float cj, lsv, lim; uint32_t inv2; };
    auto set_ones = [&](uint32_t inv2) __attribute__((always_inline)) {
        const uint32_t w = __builtin_amdgcn_perm(inv2, inv2, ones_sel);
        ones = __builtin_bit_cast(f16x8, make_uint4(w, w, w, w));
        asm volatile("" : "+v"(ones));                      // (four registers, and not copies in front of every use)
    };
    auto lane_f32 = [&](float v, int c) __attribute__((always_inline)) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), c - wbase)); };
    auto tile_info = [&](int c) __attribute__((always_inline)) {
        return TileInfo{FP8 ? lane_f32(d_cj, c) : c_exp, lane_f32(d_lv, c), lane_f32(d_lim, c), (uint32_t)__builtin_amdgcn_readlane(d_inv2, c - wbase)};
    };

    // ---- pieces of a step
    struct KFrag { i32x4 w[FP8 ? 2 : 4]; };
    struct VFrag { f16x8 f[2][2]; };                    // [16-key step][channel half]
    KFrag kf;
    VFrag vf[2];                                        // by half of the tile
    f16x8 w[2][2];                                      // fp16 weights of a group's last unit [group][16-key step]
    f32x16 sacc[2];
    int hot = 0, plain = 0;                             // tiles to prescan after a repair; those in front of `plain` need none
    auto load_kfrag = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < (FP8 ? 2 : 4); ++s) kf.w[s] = *(const i32x4 *)(lds + (slot + koff[s]));
    };
    auto load_vfrag = [&](int b, int vbase, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int ss = 0; ss < 2; ++ss)
#pragma unroll
            for (int e = 0; e < 2; ++e) vf[b].f[ss][e] = *(const f16x8 *)(lds + e * 32 * 128 + (vbase + (voff[ss] ^ (half << 6))));
    };
    auto s_product = [&](int r, int st, const f32x16 &acc, const KFrag &kf) __attribute__((always_inline)) {
        if constexpr (FP8) {
            i32x8 k8;
            k8[0] = kf.w[0][0]; k8[1] = kf.w[0][1]; k8[2] = kf.w[0][2]; k8[3] = kf.w[0][3];
            k8[4] = kf.w[1][0]; k8[5] = kf.w[1][1]; k8[6] = kf.w[1][2]; k8[7] = kf.w[1][3];
            return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(k8, q8[r], acc, 0, 0, 0, 0, 0, 0);
        } else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf.w[st]), qf[r][st], acc, 0, 0, 0);
    };
    auto products = [&](int r, const KFrag &k) __attribute__((always_inline)) {
        f32x16 s = zero16;
#pragma unroll
        for (int st = 0; st < (FP8 ? 1 : 4); ++st) s = s_product(r, st, s, k);
        return s;
    };
    auto compute_S = [&](int r) __attribute__((always_inline)) { return products(r, kf); };
    // row sums of the unit whose weights are in w[r]
    auto add_rows = [&](int r, int ss) __attribute__((always_inline)) { lsum[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, w[r][ss], lsum[r], 0, 0, 0); };
    // O^T += V^T P^T of a unit
    auto accumulate = [&](int r, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int ss = 0; ss < 2; ++ss)
#pragma unroll
            for (int e = 0; e < 2; ++e) oacc[r][e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[half].f[ss][e], w[r][ss], oacc[r][e], 0, 0, 0);
    };
    // After the step of a unit of group r (half `half` of tile t in key block j), in front of the products that consume its weights:
    // weights far above the reference, beyond the range of fp16 even, or NaN, show in the unit's row sums, and so does a ragged tile.  That
    // is the overflow check (a subtraction and a comparison a unit, where a maximum over the exponents takes ten instructions); when
    // it fires S^T is formed once more from the keys in global memory, the running maximum raised to the exact maximum over the unit
    // (accumulators and row sums are rescaled), and the weights and their sums are formed again: keys past the end of a ragged block get
    // no weight, its row sums are formed in fp32 from weights without the V scale.  A row with a NaN or +inf among its logits, or with
    // logits so large that the differences to their maximum round to more than a weight can hold, comes out NaN and must not touch
    // the others (0 NaN = NaN in the row sums on the matrix unit): its weights become zeros and its sum remembers.
    // The reference of group r raised to `top` where that is finite and above it; what the accumulators were multiplied by
    auto raise = [&](int r, float top) __attribute__((always_inline)) {
        const float m_new = top < INFINITY ? fmaxf(m_run[r], top) : m_run[r];
        const float lower = fast_exp2(m_run[r] - m_new), alpha = m_new == m_run[r] ? 1.0f : lower;
        m_run[r] = m_new;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int x = 0; x < 16; ++x) oacc[r][e][x] *= alpha;
        return alpha;
    };
    // A spoilt row stays NaN whatever follows: without its Q it raises no more alarms
    auto forget = [&](int r, bool spoilt) __attribute__((always_inline)) {
        if constexpr (FP8) {
#pragma unroll
            for (int v = 0; v < 8; ++v) q8[r][v] = spoilt ? 0 : q8[r][v];
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                uint4 q = __builtin_bit_cast(uint4, qf[r][v]);
                q.x = spoilt ? 0u : q.x; q.y = spoilt ? 0u : q.y; q.z = spoilt ? 0u : q.z; q.w = spoilt ? 0u : q.w;
                qf[r][v] = __builtin_bit_cast(bf16x8, q);
            }
        }
    };
    // (kf is lost.)
    auto repair = [&](int r, uint32_t j, int half, const TileInfo &t) __attribute__((always_inline)) {
        const int ln = lane_now(), rows = (int)j == ragged_j ? tail_rows : kBK;
        const uint8_t *row = Kh + (uint64_t)j * ktile_bytes + (uint32_t)min(32 * half + (ln & 31), rows - 1) * (uint32_t)krowb + 16 * (FP8 ? 2 : 1) * (ln >> 5);
#pragma unroll
        for (int s = 0; s < (FP8 ? 2 : 4); ++s) kf.w[s] = *(const i32x4 *)(row + (FP8 ? 16 : 32) * s);
        f32x16 s = compute_S(r);
        const int left = rows - 32 * half - 4 * (ln >> 5);
#pragma unroll
        for (int x = 0; x < 16; ++x) s[x] = 8 * (x >> 2) + (x & 3) < left ? s[x] : -INFINITY;
        const float mx = pair_max_nan(max16_nan(s)), top = mx * t.cj + t.lsv;      // -inf if the lane's row sees no real key in this unit
        const float alpha = raise(r, top), m_new = m_run[r];
        const bool special = t.inv2 == kNaN2;
        float sum = 0.f;                                    // weights without the V scale
        if (special) {
#pragma unroll
            for (int x = 0; x < 16; ++x) sum += fast_exp2(fmaf(s[x], t.cj, -m_new));
            sum = pair_sum(sum);
        }
        const bool spoilt = !(fmaf(mx, t.cj, t.lsv - m_new) <= kSpoilt) || !(sum < INFINITY);
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            const float e = fast_exp2(fmaf(s[x], t.cj, t.lsv - m_new));
            s[x] = spoilt ? 0.f : e;
        }
        w[r][0] = pack8_f16(s, 0);
        w[r][1] = pack8_f16(s, 8);
        l_full[r] = spoilt ? __builtin_nanf("") : fmaf(l_full[r], alpha, sum);
        lsum[r] = f32x4{l_old[r][0] * alpha, FP8 ? l_old[r][1] * alpha : 0.f, 0.f, 0.f};
        forget(r, spoilt);
        if (!special) { hot = kHot; plain = 0; }
        const uint32_t o = special ? 0u : __builtin_amdgcn_perm(t.inv2, t.inv2, ones_sel);
        const f16x8 own = __builtin_bit_cast(f16x8, make_uint4(o, o, o, o));
#pragma unroll
        for (int ss = 0; ss < 2; ++ss) lsum[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(own, w[r][ss], lsum[r], 0, 0, 0);
    };
    // In front of the units of a tile that is not ragged: the exact maximum over all of it, and the reference raised to that where weights
    // would pass 2^kAhead.  Of a tile whose V scale is far from the list's (inv2 = 0) also the row sums, in fp32 from weights without the
    // scale.  kslot: K slot of the tile's second half (KS = 1; the first is in kf).
    auto prescan = [&](const TileInfo &t, int kslot) __attribute__((always_inline)) {
        KFrag k2;
        if constexpr (KS == 1) {
#pragma unroll
            for (int s = 0; s < (FP8 ? 2 : 4); ++s) k2.w[s] = *(const i32x4 *)(lds + (kslot + koff[s]));
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            float mx = max16_nan(r == A ? sacc[A] : compute_S(B));
            if (KS == 1) mx = __builtin_elementwise_maximum(mx, max16_nan(products(r, k2)));
            mx = pair_max_nan(mx);
            const float top = mx * t.cj + t.lsv;
            if (__ballot(!(top <= m_run[r] + kAhead))) {
                const float alpha = raise(r, top);
                const bool spoilt = !(fmaf(mx, t.cj, t.lsv - m_run[r]) <= kSpoilt);
#pragma unroll                                              // (B's last unit is still to be added)
                for (int x = 0; x < 16; ++x) w[r][x >> 3][x & 7] = (_Float16)((float)w[r][x >> 3][x & 7] * alpha);
                l_full[r] = spoilt ? __builtin_nanf("") : l_full[r] * alpha;
                lsum[r][0] *= alpha;
                if (FP8) lsum[r][1] *= alpha;
                if (r == A) {
#pragma unroll
                    for (int x = 0; x < 16; ++x) sacc[A][x] = spoilt ? -INFINITY : sacc[A][x];
                }
                forget(r, spoilt);
                hot = kHot;
            }
            if (t.inv2 == 0u) {                             // the sums without the V scale
                float sum = 0.f;
#pragma unroll
                for (int h = 0; h < (KS == 1 ? 2 : 1); ++h) {
                    const f32x16 s = h ? products(r, k2) : r == A ? sacc[A] : compute_S(B);
#pragma unroll
                    for (int x = 0; x < 16; ++x) sum += fast_exp2(fmaf(s[x], t.cj, -m_run[r]));
                }
                l_full[r] += pair_sum(sum);
            }
        }
    };
    auto needs_repair = [&](int r, const TileInfo &t) __attribute__((always_inline)) { return __ballot(!(lsum[r][0] - l_old[r][0] <= t.lim)) != 0; };

    // ---- prologue: the first copies, the scales, Q
    if (k == 0) request_epilogue(0);
    uint32_t j_nxt = entry_j(0);                           // the key block whose second half (KS = 2: V^T tile) is asked for next
    if (k > 0) {
        request_K(k_descriptor(j_nxt, 0), 0);
        if (T::WAVES == 2) request_K(k_descriptor(j_nxt, 1), T::KSLICE);
        request_tile(v_descriptor(j_nxt), lds_v);
    }
    if (k > 1) {
        j_nxt = entry_j(1);
        request_K(k_descriptor(j_nxt, 0), 2 * T::KSLICE);
        if (KS == 2 && T::WAVES == 2) request_K(k_descriptor(j_nxt, 1), 3 * T::KSLICE);
    }
    SLA_TP(62, 2);
    const float lv_first = lvh[d_j], sk_first = FP8 ? sK[bh * Nkb + d_j] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
    // (The Q rows last: in front of the copies they would hold those up, and nothing needs them earlier.)
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int q = q0w + 32 * (r ^ kh) + l32;
        if (FP8) {
            uint4 w0 = make_uint4(0, 0, 0, 0), w1 = w0;
            if (q < N) {
                const uint8_t *qr = (const uint8_t *)Qp + head + (size_t)q * rm.ts + 32 * g;
                w0 = *(const uint4 *)qr;
                w1 = *(const uint4 *)(qr + 16);
            }
            q8[r][0] = w0.x; q8[r][1] = w0.y; q8[r][2] = w0.z; q8[r][3] = w0.w; q8[r][4] = w1.x; q8[r][5] = w1.y; q8[r][6] = w1.z; q8[r][7] = w1.w;
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                uint4 w = make_uint4(0, 0, 0, 0);
                if (q < N) w = *(const uint4 *)((const uint16_t *)Qp + head + (size_t)q * rm.ts + 16 * s + 8 * g);
                qf[r][s] = __builtin_bit_cast(bf16x8, w);
            }
        }
    }
    SLA_TP(62, 3);
    // Q, the scales and the first tiles land here, once (a builtin, so that the compiler's bookkeeping sees it)
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
    window_scales(true, lv_first, exp_constant(sk_first));
    wait_copies_and_barrier();
    SLA_TP(62, 4);
    w[A][0] = w[A][1] = w[B][0] = w[B][1] = __builtin_bit_cast(f16x8, make_uint4(0, 0, 0, 0));
#pragma unroll
    for (int x = 0; x < 4; ++x) vf[1].f[x >> 1][x & 1] = w[A][0];       // (finite: the first step multiplies them by weights of zero)
    set_ones(0u);
    if (KS == 2) vf[0] = vf[1];
    TileInfo t_cur = tile_info(0), t_prv = t_cur, t_nxt;
    uint32_t j_prv = 0;
    // S^T of A's first unit.  The reference of both groups starts as the exact maximum over their first unit (a ragged tile sets it in
    // repair), KS = 1: over their first two: with one the error against 64 bits was 1 to 3 % larger, as the largest weight of a row is then
    // less often the reference itself, a weight of exactly 1.  (KS = 2: two waves have a first unit each.)
    f32x16 second[2] = {zero16, zero16};
    if (KS == 1) {
        load_kfrag(T::KSLICE);
#pragma unroll
        for (int r = 0; r < 2; ++r) second[r] = compute_S(r);
    }
    load_kfrag(0);                                         // (an empty list multiplies what the slot holds, for nothing)
    sacc[A] = compute_S(A);
    if (t_cur.inv2 != kNaN2) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            float mx = max16_nan(r == A ? sacc[A] : compute_S(B));
            if (KS == 1) mx = __builtin_elementwise_maximum(mx, max16_nan(second[r]));
            const float top = pair_max_nan(mx) * t_cur.cj + t_cur.lsv;
            m_run[r] = top < INFINITY ? fmaxf(m_run[r], top) : m_run[r];
        }
    }

    SLA_TP(62, 5);
#define SLA_SB() __builtin_amdgcn_sched_barrier(0)
#define SLA_PIN(...) asm volatile("" : __VA_ARGS__)
    // Step of group X (see above) in issue order (one MFMA, then a staggered share of the vector
    // work, held in place by data dependencies and scheduling barriers), X's unit being half `half` of tile t.  (jy, halfy, ty): the
    // other group's last unit.  kslot: K slot of the next slice, whose fragments step A reads and step B holds; vslot: V^T slot of X's unit,
    // whose fragments step A reads.
    auto step = [&](auto xc, int b, const TileInfo &t, uint32_t jy, int halfy, const TileInfo &ty, int kslot, int vslot, int half) __attribute__((always_inline)) {
        constexpr int X = decltype(xc)::value, Y = X ^ 1;
        f32x16 sn = zero16;
        f32x16 &s = sacc[X];
        uint32_t pw[8];
        float moff = t.lsv - m_run[X];
        auto pv = [&](int ss, int e) { oacc[Y][e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[X == A ? b ^ 1 : b].f[ss][e], w[Y][ss], oacc[Y][e], 0, 0, 0); };
        auto sm = [&](int st) { sn = s_product(Y, st, sn, kf); };
        auto fm = [&](int x0, int x1) {
#pragma unroll
            for (int x = x0; x <= x1; ++x) s[x] = fmaf(s[x], t.cj, moff);
        };
        auto ex = [&](int x0, int x1) {
#pragma unroll
            for (int x = x0; x <= x1; ++x) s[x] = fast_exp2(s[x]);
        };
        auto cv2 = [&](int pr) { pw[pr] = pack_f16(s[2 * pr], s[2 * pr + 1]); };
        auto mend = [&]() __attribute__((always_inline)) {                   // (behind the products that read kf)
            if (__builtin_expect(needs_repair(Y, ty), 0)) {
                repair(Y, jy, halfy, ty);
                if constexpr (X == B) load_kfrag(kslot);
            }
            if constexpr (X == A) load_kfrag(kslot);
        };
        SLA_SB();
        if constexpr (X == A) load_vfrag(b, vslot, half);
        l_old[Y][0] = lsum[Y][0];
        if (FP8) l_old[Y][1] = lsum[Y][1];
        if (!FP8) {
            sm(0);          fm(0, 2);   ex(0, 0);
            SLA_PIN("+v"(sn), "+v"(moff)); SLA_SB();
            add_rows(Y, 0); ex(1, 1);   fm(3, 4);
            SLA_PIN("+v"(lsum[Y]), "+v"(moff)); SLA_SB();
            sm(1);          ex(2, 3);   cv2(0);     fm(5, 6);
            SLA_PIN("+v"(sn), "+v"(moff), "+v"(pw[0])); SLA_SB();
            add_rows(Y, 1); ex(4, 4);
            SLA_PIN("+v"(lsum[Y]), "+v"(moff)); SLA_SB();
            sm(2);          ex(5, 5);   cv2(1);     ex(6, 6);   fm(7, 8);
            SLA_PIN("+v"(sn), "+v"(moff), "+v"(pw[1])); SLA_SB();
            sm(3);          ex(7, 7);   cv2(2);     fm(9, 10);  ex(8, 8);
            SLA_PIN("+v"(sn), "+v"(moff), "+v"(pw[2]), "+v"(s)); SLA_SB();
            mend();
            pv(0, 0);       cv2(3);     ex(9, 10);  fm(11, 12);
            SLA_PIN("+v"(oacc[Y][0]), "+v"(moff), "+v"(pw[3])); SLA_SB();
            pv(0, 1);       cv2(4);     ex(11, 12); fm(13, 14);
            SLA_PIN("+v"(oacc[Y][1]), "+v"(moff), "+v"(pw[4])); SLA_SB();
            pv(1, 0);       cv2(5);     ex(13, 14); fm(15, 15);
            SLA_PIN("+v"(oacc[Y][0]), "+v"(pw[5])); SLA_SB();
            pv(1, 1);       ex(15, 15); cv2(6);
            SLA_PIN("+v"(oacc[Y][1]), "+v"(pw[6])); SLA_SB();
        } else {
            sm(0);          SLA_SB();               // (the e4m3 MFMA takes twice as long: a larger first share)
            fm(0, 3);       ex(0, 2);   fm(4, 5);
            SLA_PIN("+v"(sn), "+v"(moff)); SLA_SB();
            add_rows(Y, 0); ex(3, 3);   cv2(0);
            SLA_PIN("+v"(lsum[Y]), "+v"(moff), "+v"(pw[0])); SLA_SB();
            add_rows(Y, 1); ex(4, 5);   cv2(1);     fm(6, 8);
            SLA_PIN("+v"(lsum[Y]), "+v"(moff), "+v"(pw[1]), "+v"(s)); SLA_SB();
            mend();
            pv(0, 0);       cv2(2);     ex(6, 7);   fm(9, 10);
            SLA_PIN("+v"(oacc[Y][0]), "+v"(moff), "+v"(pw[2])); SLA_SB();
            pv(0, 1);       cv2(3);     ex(8, 9);   fm(11, 12);
            SLA_PIN("+v"(oacc[Y][1]), "+v"(moff), "+v"(pw[3])); SLA_SB();
            pv(1, 0);       cv2(4);     ex(10, 12); fm(13, 14);
            SLA_PIN("+v"(oacc[Y][0]), "+v"(moff), "+v"(pw[4])); SLA_SB();
            pv(1, 1);       cv2(5);     ex(13, 14); fm(15, 15); cv2(6); ex(15, 15);
            SLA_PIN("+v"(oacc[Y][1]), "+v"(pw[5]), "+v"(pw[6])); SLA_SB();
        }
        cv2(7);
        w[X][0] = __builtin_bit_cast(f16x8, make_uint4(pw[0], pw[1], pw[2], pw[3]));
        w[X][1] = __builtin_bit_cast(f16x8, make_uint4(pw[4], pw[5], pw[6], pw[7]));
        sacc[Y] = sn;
    };
#undef SLA_PIN
    using GA = std::integral_constant<int, A>;
    using GB = std::integral_constant<int, B>;
    // Requests of iteration c (phase P): what iteration c+1 reads, or the epilogue's operands during the last tile.  (The first half of a
    // tile c+2 past the end of the list is replaced by that of the last tile, in a slot nobody reads.)
    auto requests = [&](int c, int P) __attribute__((always_inline)) {
        if (KS == 2) {
            if (c + 2 < k) {
                const uint32_t j = entry_j(c + 2);
                request_K(k_descriptor(j, 0), 2 * P * T::KSLICE);
                if (T::WAVES == 2) request_K(k_descriptor(j, 1), (2 * P + 1) * T::KSLICE);
            }
            if (c + 1 < k) {
                request_tile(v_descriptor(j_nxt), lds_v + (P ^ 1) * T::VBYTES);
                j_nxt = entry_j(min(c + 2, k - 1));
            } else request_epilogue(P);
        } else if (c + 1 < k) {
            request_K(k_descriptor(j_nxt, 1), ((2 * P + 3) & 3) * T::KSLICE);
            request_tile(v_descriptor(j_nxt), lds_v + (P ^ 1) * T::VBYTES);
            j_nxt = entry_j(min(c + 2, k - 1));
            request_K(k_descriptor(j_nxt, 0), 2 * P * T::KSLICE);
        } else request_epilogue(P);
    };
    // c: the next tile
    auto set_plain = [&](int c) __attribute__((always_inline)) {
        const unsigned long long far = d_far >> ((c - wbase) & 63);
        plain = hot > 0 ? 0 : far ? c + __builtin_ctzll(far) : k;
    };
    auto iteration = [&](int c, auto phase) __attribute__((always_inline)) {
        constexpr int P = decltype(phase)::value;
        constexpr int vslot = T::VRING + P * T::VBYTES;
        SLA_T(c, 0);
        wait_copies_and_barrier();
        SLA_T(c, 1);
        const uint32_t j_cur = entry_j(c);
        t_nxt = tile_info(min(c + 1, k - 1));
        SLA_T(c, 2);
        if (__builtin_expect(c >= plain, 0)) {
            hot -= hot > 0;
            if (t_cur.inv2 != kNaN2) prescan(t_cur, (2 * P + 1) * T::KSLICE);
            set_plain(c + 1);
        }
        if constexpr (KS == 2) {
            constexpr int k1 = 2 * (P ^ 1) * T::KSLICE;
            step(GA{}, P, t_cur, j_prv, kh, t_prv, k1, vslot, 0);
            requests(c, P);
            set_ones(t_cur.inv2);
            SLA_T(c, 3);
            step(GB{}, P, t_cur, j_cur, kh, t_cur, k1, 0, 0);
        } else {
            constexpr int k1 = (2 * P + 1) * T::KSLICE, k2 = ((2 * P + 2) & 3) * T::KSLICE;
            step(GA{}, 0, t_cur, j_prv, 1, t_prv, k1, vslot, 0);
            requests(c, P);
            set_ones(t_cur.inv2);                          // the units whose sums are formed from here on are this tile's
            step(GB{}, 0, t_cur, j_cur, 0, t_cur, k1, 0, 0);
            SLA_T(c, 3);
            step(GA{}, 1, t_cur, j_cur, 0, t_cur, k2, vslot, 1);
            step(GB{}, 1, t_cur, j_cur, 1, t_cur, k2, 0, 0);
        }
        SLA_T(c, 4);
        t_prv = t_cur; j_prv = j_cur;
        t_cur = t_nxt;
    };
    for (int c = 0; c < k;) {
        // the window: an iteration's requests reach two tiles ahead (never moves for lists of at most 64 blocks)
        if (c + 2 - wbase >= 64 && wbase + 64 < k) load_window(wbase + 32);
        const int end = k - wbase > 64 ? wbase + 62 : k;
        set_plain(c);
        do {                                               // two iterations, so that slots are constants
            iteration(c, std::integral_constant<int, 0>{});
            if (++c == end) break;
            iteration(c, std::integral_constant<int, 1>{});
            ++c;
        } while (c < end);
    }
#undef SLA_SB

    wait_copies_and_barrier();                          // epilogue operands landed; every wave is past its last tile
    const int elane = lane_now(), e32 = elane & 31, eg = elane >> 5;         // (the loop carries no lane index)
    SLA_TP(61, 0);
    l_old[B][0] = lsum[B][0];
    l_old[B][1] = lsum[B][1];
    add_rows(B, 0);
    add_rows(B, 1);
    if (__builtin_expect(needs_repair(B, t_prv), 0)) repair(B, j_prv, KS == 2 ? kh : 1, t_prv);
    const int PL = k > 0 ? (k - 1) & 1 : 0;                // phase of the last tile
    if (KS == 2) { if (PL) accumulate(B, 1); else accumulate(B, 0); } else accumulate(B, 1);                              // B's last unit
    const uint8_t *stA = lds + hq_off(PL), *stB = lds + wt_off(PL), *zrow = lds + T::ZOFF;
    uint8_t *ot = lds + T::VRING + PL * T::VBYTES + wave_u * 4096;           // the last V^T tile's slot: nobody reads it any more
    float l_run[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) l_run[r] = lsum[r][0] + (FP8 ? lsum[r][1] : 0.f) + l_full[r];
    // KS = 2: the two waves that share rows exchange a group each (accumulators, reference exponent and row sums): what a wave has of its
    // group B is the other one's A.  It is left in LDS here and taken behind the linear branch, whose arithmetic hides the way.
    // Two waves: wave 0 leaves its 8 KB in the last V^T tile's slot, wave 1 in the free part of the K ring.
    auto place = [&](int wv) -> uint8_t * {
        if (RH == 2) return lds + T::OOFF + wv * 8192;
        return wv ? lds + (FP8 ? 0 : PL ? 2 * T::KSLICE : 0) : lds + T::VRING + PL * T::VBYTES;
    };
    if constexpr (KS == 2) {
        float4 *xo = (float4 *)place(wave_u) + elane;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                xo[(4 * e + x) * 64] = make_float4(oacc[B][e][4 * x], oacc[B][e][4 * x + 1], oacc[B][e][4 * x + 2], oacc[B][e][4 * x + 3]);
        ((float2 *)(lds + T::XOFF))[64 * wave_u + elane] = make_float2(m_run[B], l_run[B]);
        ot = place(wave_u ^ 1);                            // (what this wave alone reads; the transposed store goes through it)
    }
    constexpr int GROUPS = KS == 2 ? 1 : 2;                // groups this wave finishes
#pragma unroll
    for (int r = 0; r < GROUPS; ++r) {
        f32x16 lin[2] = {zero16, zero16};                  // the linear branch, projected
        if (r == 0) SLA_TP(61, 1);
        if (Hq != nullptr) {
            bf16x8 hfr[4][2], wfr[4][2];                   // read in one go: their latency passes behind the arithmetic of phi(Q)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int hchunk = FP8 ? 4 * eg + s : 2 * s + eg;      // 16-byte chunk holding channels dcol(s)..dcol(s)+7
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    hfr[s][e] = *(const bf16x8 *)(stA + (32 * e + e32) * 128 + ((hchunk ^ swz8(e32)) << 4));
                    wfr[s][e] = *(const bf16x8 *)(stB + (32 * e + e32) * 128 + (((2 * s + eg) ^ swz8(e32)) << 4));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---- phi(Q): x[8s + c] is channel dcol(s) + c, the channel slot c of K-step s carries in the product below
            float x[32];
            if (FP8) {
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(q8[r][v], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(q8[r][v], true);
                    x[4 * v + 0] = lo[0] * qscale; x[4 * v + 1] = lo[1] * qscale; x[4 * v + 2] = hi[0] * qscale; x[4 * v + 3] = hi[1] * qscale;
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint4 v = __builtin_bit_cast(uint4, qf[r][s]);
                    x[8 * s + 0] = bf16_lo(v.x); x[8 * s + 1] = bf16_hi(v.x);
                    x[8 * s + 2] = bf16_lo(v.y); x[8 * s + 3] = bf16_hi(v.y);
                    x[8 * s + 4] = bf16_lo(v.z); x[8 * s + 5] = bf16_hi(v.z);
                    x[8 * s + 6] = bf16_lo(v.w); x[8 * s + 7] = bf16_hi(v.w);
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
            } else {                                       // ELU(x)+1, elementwise
#pragma unroll
                for (int d = 0; d < 32; ++d) x[d] = x[d] > 0.f ? x[d] + 1.0f : fast_exp2(x[d] * kLog2e);
            }
            bf16x8 fq[4];
            float den = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int dcol = FP8 ? 32 * eg + 8 * s : 16 * s + 8 * eg;
                uint4 o;
                o.x = pack_bf16(x[8 * s + 0] * inv, x[8 * s + 1] * inv); o.y = pack_bf16(x[8 * s + 2] * inv, x[8 * s + 3] * inv);
                o.z = pack_bf16(x[8 * s + 4] * inv, x[8 * s + 5] * inv); o.w = pack_bf16(x[8 * s + 6] * inv, x[8 * s + 7] * inv);
                fq[s] = __builtin_bit_cast(bf16x8, o);
                const uint4 z = *(const uint4 *)(zrow + dcol * 2);
                den = dot2_bf16(o.w, z.w, dot2_bf16(o.z, z.z, dot2_bf16(o.y, z.y, dot2_bf16(o.x, z.x, den))));
            }
            den += xchg32(den);
            const float inv_den = den > 0.f ? 1.0f / den : 0.f;     // no marginal block: H = Z = 0 and O_lin = 0

            if (r == 0) SLA_TP(61, 2);
            // ---- O_lin^T = Hq^T phi(Q)^T, then W^T O_lin^T
            f32x16 lacc[2];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int e = 0; e < 2; ++e) lacc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hfr[s][e], fq[s], s == 0 ? zero16 : lacc[e], 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int y = 0; y < 16; ++y) lacc[e][y] *= inv_den;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bf16x8 pf = pack8(lacc[s >> 1], 8 * (s & 1));
#pragma unroll
                for (int e = 0; e < 2; ++e) lin[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfr[s][e], pf, s == 0 ? zero16 : lin[e], 0, 0, 0);
            }
        }
        // ---- normalise the sparse output (the weights carried the V scale relative to the list's reference) and add the two
        f32x16 (&o)[2] = oacc[r];
        float l = l_run[r], own = 1.f, given = 0.f;
        float4 in[2][4];
        if constexpr (KS == 2) {
            lds_barrier();
            const float2 ml = ((const float2 *)(lds + T::XOFF))[64 * (wave_u ^ 1) + elane];
            const float4 *xi = (const float4 *)place(wave_u ^ 1) + elane;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int x = 0; x < 4; ++x) in[e][x] = xi[(4 * e + x) * 64];
            const float m = fmaxf(m_run[A], ml.x);
            own = fast_exp2(m_run[A] - m);
            given = fast_exp2(ml.x - m);
            l = fmaf(l, own, ml.y * given);
        }
        const float inv_l = l > 0.f ? fast_exp2(lv_ref) / l : l;     // 0 for an empty list, NaN for a spoilt row
        own *= inv_l;
        given *= inv_l;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                o[e][x] = fmaf(o[e][x], own, lin[e][x]);
                if constexpr (KS == 2) o[e][x] = fmaf(((const float *)&in[e][x >> 2])[x & 3], given, o[e][x]);
            }
        if (r == 0) SLA_TP(61, 3);
        // ---- store.  Register 4a+b of oacc[r][e] is channel 32e + 8a + 4g + b of the row: the 32x64 tile is transposed through
        // the wave's own 4 KB of LDS (8-byte pieces, XOR-swizzled by row) so that it leaves as full rows, 16 bytes per lane.
        const int qr = q0w + 32 * (r ^ kh);
        if (O32 != nullptr) {                              // diagnostic output: the fp32 values the bf16 store would round
            if (qr + e32 < N) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int aa = 0; aa < 4; ++aa)
                        *(float4 *)(O32 + head + (size_t)(qr + e32) * rm.ts + 32 * e + 8 * aa + 4 * eg) =
                            make_float4(oacc[r][e][4 * aa + 0], oacc[r][e][4 * aa + 1], oacc[r][e][4 * aa + 2], oacc[r][e][4 * aa + 3]);
            }
        } else {
            const int f = ((e32 >> 1) & 7) << 1;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int aa = 0; aa < 4; ++aa) {
                    uint2 o;
                    o.x = pack_bf16(oacc[r][e][4 * aa + 0], oacc[r][e][4 * aa + 1]);
                    o.y = pack_bf16(oacc[r][e][4 * aa + 2], oacc[r][e][4 * aa + 3]);
                    const int piece = 8 * e + 2 * aa + eg;
                    *(uint2 *)(ot + e32 * 128 + ((piece ^ f) << 3)) = o;
                }
            wave_lds_sync();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int row = 8 * kk + (elane >> 3), ch = elane & 7;       // row of the tile, 16-byte chunk of the row
                const int fr = ((row >> 1) & 7) << 1;
                const uint4 v = *(const uint4 *)(ot + row * 128 + (((2 * ch) ^ fr) << 3));
                if (qr + row < N) *(uint4 *)(O + head + (size_t)(qr + row) * rm.ts + ch * 8) = v;
            }
            if (r == 0) SLA_TP(61, 4);
            wave_lds_sync();                               // (the second group's tile takes the same place)
        }
    }
    SLA_TP(61, 5);
#ifdef SLA_PROBE_TIME
    if (threadIdx.x == 0 && work < 32768) sla_wg_times[2 * work + 1] = __builtin_amdgcn_s_memrealtime();
    if (probe_on) {
        const unsigned long long tp_c1 = __builtin_readcyclecounter(), tp_r1 = __builtin_amdgcn_s_memrealtime();
        if (lane == 0) { tprobe[63 * 8 + 6] = tp_c1 - tp_c0; tprobe[63 * 8 + 7] = tp_r1 - tp_r0; }   // wave life: shader clock, 100 MHz clock
        for (int x = lane; x < 64 * 8; x += 64) sla_probe_times[x] = tprobe[x];
    }
#endif
}

// W [nW][e_in][e_out] -> WT [nW][e_out][slot] as its own launch (the whole forward folds this into the states pass)
__global__ __launch_bounds__(256) void transpose_w_kernel(const uint16_t *__restrict__ W, uint16_t *__restrict__ WT)
{
    transpose_w_tile(W + (size_t)blockIdx.x * kD * kD, WT + (size_t)blockIdx.x * kD * kD, 256);
}

#ifdef SLA_PROBE_TIME
extern "C" int sla_probe_read_wg(unsigned long long *dst, int n) { return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(sla_wg_times), sizeof(unsigned long long) * 2 * n); }
extern "C" int sla_probe_read(unsigned long long *dst) { return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(sla_probe_times), sizeof(unsigned long long) * 64 * 8); }
#endif

hipError_t launch_transpose_w(const void *W, int nW, void *WT, hipStream_t st)
{
    transpose_w_kernel<<<nW, 256, 0, st>>>((const uint16_t *)W, (uint16_t *)WT);
    return hipGetLastError();
}

// Whether the keys of a 128-row query block are split between waves as well: four waves, twice the speed per block, two blocks to a CU
// where the two-wave form has four.  It pays where that saves half a round, in the first half of the two-wave form's first round and of
// its second; from the third on the dispatch of blocks evens the rounds out.  Layers of 16 heads, split / not, us, bf16 lists of 3 %, 10 % and 20 %
// of the blocks, then E4M3: 480 blocks 33.1 / 34.5, 38.0 / 41.1, 44.3 / 50.1; 37.0 / 39.1, 40.9 / 44.8, 46.6 / 53.2; 576 blocks 39.6 / 38.3, 46.8 / 45.3,
// 57.3 / 55.0; 40.8 / 39.4, 46.4 / 45.0, 56.2 / 54.9; 896: 47.8 / 45.2, 63.1 / 59.6, 86.1 / 81.0; 44.5 / 42.5, 58.5 / 55.2, 78.0 / 72.8; 1120: 62.9 / 61.7,
// 88.0 / 88.4, 125 / 128; 59.7 / 58.9, 81.3 / 82.3, 114 / 117; 1520: 78.6 / 80.3, 120 / 127, 181 / 195; 73.1 / 74.7, 109 / 117, 160 / 173; at 5 %
// 1552: 101 / 99; 94 / 91; 2400: 177 / 167; 155 / 146.
// (The two forms add in another order: with 128-row blocks the last bits of a head can depend on how many blocks the launch has.)
static bool split_keys(long total)
{
    constexpr long kSlots = 4 * 256;                       // workgroups of the two-wave form the chip holds
    return total <= kSlots / 2 || (total > kSlots && total <= 3 * kSlots / 2);
}

hipError_t launch_attend(const void *Q, const void *K, const void *Vp, const float *lvs,
                         const float *sQ, const float *sK, bool fp8, RowMap rm,
                         const int32_t *crit_idx, int k_c, const void *Hq, const void *WT,
                         int proj_per_head, int phi, int B, int H, int N, int bq, float sm_scale,
                         void *O, float *O32, hipStream_t st)
{
    const int Nqb = (N + bq - 1) / bq, Nkb = (N + kBK - 1) / kBK;
    const long total = (long)B * H * Nqb;
    const float c_exp = sm_scale * kLog2e;
    auto go = [&](auto kernel, int threads) {
        kernel<<<(unsigned)xcd_grid(total), threads, 0, st>>>(Q, K, (const uint16_t *)Vp, lvs, sQ, sK, rm, crit_idx, k_c, (const uint16_t *)Hq, (const uint16_t *)WT,
                                                          proj_per_head, phi, H, N, Nqb, Nkb, total, c_exp, (uint16_t *)O, O32);
        return hipGetLastError();
    };
    if (bq == 128) {
        if (split_keys(total)) return fp8 ? go(attend_kernel<true, 2, 2>, 256) : go(attend_kernel<false, 2, 2>, 256);
        return fp8 ? go(attend_kernel<true, 2, 1>, 128) : go(attend_kernel<false, 2, 1>, 128);
    }
    // lists of at most two blocks (frame attention): the kernel without a pipeline, eight workgroups per CU
    if (k_c <= kShortList) return go(attend_short_kernel_for(fp8), 128);
    return fp8 ? go(attend_kernel<true, 1, 2>, 128) : go(attend_kernel<false, 1, 2>, 128);
}

}  // namespace sla
