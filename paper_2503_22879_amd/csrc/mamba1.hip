// The 8-bit Mamba1 selective scan (Section 3.2, Eq. 2 in the Mamba1 parameterisation; the framework's 8-bit
// selective-scan kernel of Section 4.2): per sequence b, channel d, state n
//     h_t[d,n] = exp(Delta_t[d] A[d,n]) h_{t-1}[d,n] + Delta_t[d] B_t[n] x_t[d],   y_t[d] = sum_n C_t[n] h_t[d,n] + D[d] x_t[d]
// on int8 x (one scale per channel range), int8 B and C (one scale each).  Tensors are channel-major with time last:
// x, Delta, y [b, D, L]; B, C [b, N, L]; A [D, N]; states [b, D, N].
//
// There is no contraction to put on the matrix cores: every (token, channel, state) element needs its own
// exponential, so the kernel is bound by the vector ALU and is organised to keep that unit busy.  A group of LPC lanes owns
// one channel at a time and a tile of 16 LPC tokens, 16 consecutive tokens per lane: per state it forms the 16 decay
// factors and inputs of its tokens, reduces them to one (product, state) pair, scans the pairs over the group's lanes with
// data-parallel-primitive row shifts and broadcasts (the operator of a first-order linear recurrence), and replays its 16
// tokens from the scanned-in state while accumulating y.  The tile's B and C sit in LDS, shared by the channels of the
// workgroup; the state at the end of a tile is carried to the next tile through LDS.
#include <algorithm>

#include "quamba_internal.h"

namespace quamba {
namespace {

constexpr int kE = 16;              // tokens per lane
constexpr float kLog2e = 1.44269504088896340736f;
constexpr int kDecodeSeqs = 4;      // sequences per thread and trip of the decode step
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_fetch(float old, float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v),
                                                                 CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Inclusive scan of (P, h) pairs over groups of LPC lanes (16, 32 or 64).  One step applies the pair fetched from an earlier lane first and
// the lane's own after it: (Ps, hs) then (P, h) -> (Ps P, P hs + h), as two instructions whose first source is the
// shifted lane: h += hs * P, then P *= Ps.  Lanes without a source lane (and rows the mask leaves out) are not
// written, which is the identity.  Shifts by 1, 2, 4, 8 inside rows of 16 lanes, then lane 15 of rows 0 and 2 into
// rows 1 and 3, then lane 31 into rows 2 and 3.  The two idle cycles in front of each step are the wait a
// data-parallel-primitive read needs after a vector write of the same register.
#define QUAMBA_SCAN_STEP(ctrl)                                                       \
    "s_nop 1\n\t"                                                                    \
    "v_fmac_f32_dpp %0, %0, %1 " ctrl " bank_mask:0xf\n\t"                           \
    "v_mul_f32_dpp %1, %1, %1 " ctrl " bank_mask:0xf\n\t"
#define QUAMBA_SCAN_ROW                                                                            \
    "s_setprio 2\n\t" QUAMBA_SCAN_STEP("row_shr:1 row_mask:0xf") QUAMBA_SCAN_STEP("row_shr:2 row_mask:0xf") \
    QUAMBA_SCAN_STEP("row_shr:4 row_mask:0xf") QUAMBA_SCAN_STEP("row_shr:8 row_mask:0xf")
template <int LPC>
__device__ __forceinline__ void wave_scan(float &P, float &h)
{
    if (LPC == 16)
        asm volatile(QUAMBA_SCAN_ROW "s_nop 1\n\ts_setprio 0" : "+v"(h), "+v"(P));
    else if (LPC == 32)
        asm volatile(QUAMBA_SCAN_ROW QUAMBA_SCAN_STEP("row_bcast:15 row_mask:0xa") "s_nop 1\n\ts_setprio 0"
                     : "+v"(h), "+v"(P));
    else
        asm volatile(QUAMBA_SCAN_ROW QUAMBA_SCAN_STEP("row_bcast:15 row_mask:0xa")
                     QUAMBA_SCAN_STEP("row_bcast:31 row_mask:0xc") "s_nop 1\n\ts_setprio 0"
                     : "+v"(h), "+v"(P));
}
#undef QUAMBA_SCAN_ROW
#undef QUAMBA_SCAN_STEP

// log(1 + exp(v)) = max(v, 0) + log(1 + e), e = exp(-|v|), on the hardware's base-2 exponential and logarithm, with what
// the roundings in front of each drop put back: of the product |v| log2 e (which would cost e |v| units of 2^-24) and of the
// sum 1 + e (which would cost the logarithm 2^-24 / e of its value, 2e-6 at e = 1/32).  In error against 64 bits this is
// log1pf(expf()) of the library, which the one-thread kernel and the step use, at a third of the instructions.
__device__ __forceinline__ float softplus_fast(float v)
{
    constexpr float kLn2 = 0.69314718055994530942f, kLn2Rest = (float)(0.69314718055994530942 - (double)kLn2);
    const float w = -__builtin_fabsf(v), t = w * kLog2e;
    // exp(w) = 2^t exp(r), r = w - t ln 2; the bound only catches w = -inf, whose r is no number (2^t is 0 then)
    const float r = fmaxf(fmaf(-t, kLn2Rest, fmaf(-t, kLn2, w)), -1.0f);
    const float e0 = __builtin_amdgcn_exp2f(t), e = fmaf(e0, r, e0);
    // log(1 + e) = log(s) + lost / s; 1 - 0.6 e is 1/s to within 0.1 (at e = 1) and is 1 to within e / 2 for small e,
    // which leaves less than 2^-25 of the result
    const float s = 1.0f + e, lost = e - (s - 1.0f);
    return fmaxf(v, 0.0f) + fmaf(__builtin_amdgcn_logf(s), kLn2, fmaf(-0.6f * e, lost, lost));
}

__device__ __forceinline__ float byte_to_float(uint32_t w, int k) { return (float)(int)(int8_t)(w >> (8 * k)); }

// 2^x of 17 values at raised wave priority.  A SIMD issues plain fp32 instructions of two waves at once, but an exponential
// blocks it for 8 cycles.  With the exponentials of its waves scattered between the others' plain instructions the pairing
// hardly ever happens; as uninterrupted bursts they leave stretches in which it does (a loop of 16 exponentials and 80
// multiply-adds, 4 waves per SIMD: 192 ns per turn and SIMD, with the bursts prioritised 143).
__device__ __forceinline__ void exp2_burst(float (&v)[kE], float &p)
{
#define QUAMBA_E(i) "v_exp_f32 %" #i ", %" #i "\n\t"
    asm volatile("s_setprio 2\n\t"
                 QUAMBA_E(0) QUAMBA_E(1) QUAMBA_E(2) QUAMBA_E(3) QUAMBA_E(4) QUAMBA_E(5) QUAMBA_E(6) QUAMBA_E(7) QUAMBA_E(8)
                 QUAMBA_E(9) QUAMBA_E(10) QUAMBA_E(11) QUAMBA_E(12) QUAMBA_E(13) QUAMBA_E(14) QUAMBA_E(15) QUAMBA_E(16)
                 "s_setprio 0\n\ts_nop 0"  // also the wait a use of an exponential's result needs
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]),
                   "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]), "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15]),
                   "+v"(p));
#undef QUAMBA_E
}

// 16 bytes / 4 floats / 8 halves at any byte resp. element address: the hardware takes unaligned vector accesses, so a
// row may start anywhere (a sequence length that is no multiple of 16 shifts every row).
typedef u32x4 u32x4_u __attribute__((aligned(1)));
typedef u32x4 u32x4_f __attribute__((aligned(4)));
typedef u32x4 u32x4_h __attribute__((aligned(2)));

// The 16 codes of tokens t .. t + 15 of a row of L >= 16; those past the end are zero and are not read: a lane that would
// cross the end reads the row's last 16 codes and shifts.
__device__ __forceinline__ u32x4 load_codes(const int8_t *row, int t, int L)
{
    const int t1 = min(t, L - kE), k = t - t1;
    u32x4 v = *reinterpret_cast<const u32x4_u *>(row + t1);
    if (k > 0) {
        if (k & 8) v = (u32x4){v[2], v[3], 0, 0};
        if (k & 4) v = (u32x4){v[1], v[2], v[3], 0};
        v = (u32x4){__builtin_amdgcn_alignbyte(v[1], v[0], k), __builtin_amdgcn_alignbyte(v[2], v[1], k),
                    __builtin_amdgcn_alignbyte(v[3], v[2], k), __builtin_amdgcn_alignbyte(0, v[3], k)};
        if (k >= kE) v = (u32x4){0, 0, 0, 0};
    }
    return v;
}

// A workgroup's kThreads / LPC channels of one sequence, N = 16 states, seqlen >= 16.  LPC lanes share a channel (64, 32 or 16), so a
// wave holds 64 / LPC channels.  B and C of NS states are staged at a time: 8 with workgroups of 256 threads, whose 34 KB of
// LDS let four of them share a compute unit, all 16 with 512 and 768 (8 in the halves of mamba1_scan_halves_kernel).  The loop over states stays rolled: the 16 tokens of a lane
// already give every instruction 16 independent copies, and unrolling further only costs registers.  B and C are staged as fp32 (converted once per workgroup
// instead of once per channel): plain fp32 multiplies and multiply-adds of two waves can issue together, the
// mixed-precision ones that take fp16 operands cannot.  LDS rows are [state][quarter of a lane's tokens][lane], so that a lane's
// four 16-byte reads are consecutive across the lanes.
// C is staged times its scale and the skip term starts the output's sum, so that the sum is y.  That is one more fp32
// rounding per code: 8.2e-8 instead of 7.7e-8 (rms) in the sum, under the 2e-4 of the fp16 output, whose error against 64 bits
// is the same to four digits; exact codes, with x read again for the skip term at the end, took 1 to 2 % longer.
// Measured at 4 x 4096 tokens, 5120 channels: 308 to 321 us (387 to 393 with fp16 operands, tiles of 1024
// tokens and the exponentials between the other instructions); 1003 tokens of one sequence in workgroups of 24: 28.5 us, with gate and step-size
// codes 30.6 (32 to 34 with workgroups of 8 channels, 36.5 with 512 threads, 3000 with one thread per channel, which is what a length
// that is no multiple of 16 took before).  By the counters 36 cycles of a SIMD per 64 elements; the loop's instructions take 23 where all
// plain ones of two waves issue together, 33 where none do.
template <int LPC, int kThreads, int NS, bool HALVES = false, int kTiles = 1, bool MIXED = false>
__device__ __forceinline__ void scan_channels(
    const SsdArgs &a, const float *A, const float *init, float *fin, int b, unsigned blk,  // the sequence, which kThreads / LPC of its channels
    f32x4 *s_B, f32x4 *s_C,  // [state][quarter][lane of a tile, kTiles of them]
    float2 *s_AH,            // [channel][state]: A log2(e), the state before the tile
    float *s_silu)           // SiLU(z_scale * code), by the gate code's byte
{
    constexpr int N = 16, kTile = LPC * kE, kCh = MIXED ? 20 : kThreads / LPC;  // channels of the workgroup
    constexpr int kLanes = LPC * kTiles, kStagers = kThreads / kLanes;
    constexpr bool kAlone = LPC == 64 && NS == 16 && !MIXED, kAhead = kAlone || kThreads == 768;
    // Lanes of a scan.  In mamba1_scan_halves_kernel the 64 lanes of a channel take their tile as two of 32 lanes, one after the other,
    // and groups of 32 lanes decide for themselves where a number is not finite: the same operations, bit for bit, in both parts of
    // its launch, so that equal sequences of a call have equal results.
    constexpr bool kTwo = HALVES && LPC == 64;
    constexpr int kScan = kTwo ? 32 : LPC;
    const int D = a.s.headdim, L = a.s.seqlen;
    const int sub = threadIdx.x & (LPC - 1);  // the lane inside its channel's group
    const int ch = MIXED && LPC == 64 ? 16 + (threadIdx.x - 512) / 64 : threadIdx.x / LPC;  // the channel inside the workgroup
    const int stage_lane = threadIdx.x & (kLanes - 1), stager = threadIdx.x / kLanes;
    const int d = blk * kCh + ch;
    const bool own = d < D;                   // lanes without a channel redo the last one and store nothing
    const int dd = own ? d : D - 1;
    const float sC = a.C_scales[0];
    const float sx = x_scale_lookup(a, 0, dd);
    const float sxB = sx * a.B_scales[0], Dx = (a.D ? a.D[dd] : 0.0f) * sx;

    for (int i = threadIdx.x; i < kCh * N; i += kThreads) {
        const int c = min((int)blk * kCh + i / N, D - 1), n = i % N;
        // A = -inf (a state that forgets everything) as the largest number: a token past the end has a step of 0, which must
        // not make 0 times infinity of it
        const float A2 = A[(size_t)c * N + n] * kLog2e;
        s_AH[i] = make_float2(A2 == -__builtin_inff() ? -3.402823466e38f : A2, init ? init[((size_t)b * D + c) * N + n] : 0.0f);
    }
    if (a.z)
        for (int i = threadIdx.x; i < 256; i += kThreads) s_silu[i] = silu_of_code(a.z_scale, (int8_t)i);

    // Row addresses and token indices are derived anew, from a channel and lane index the compiler must take for new ones,
    // where a tile begins and where it ends: kept across the loop over states they would take the registers that
    // let its LDS reads be requested ahead.
    auto anew = [&](int t0, size_t &row, int &t) {
        int c = dd, l = sub;
        asm volatile("" : "+v"(c), "+v"(l));
        row = ((size_t)b * D + c) * L;
        t = t0 + kE * l;
    };
    // the codes of the tile at t0, with 16 fp32 step sizes or their 16 codes in the first piece
    auto load_tile = [&](int t0, u32x4 &xq, u32x4 (&raw)[4]) {
        size_t row;
        int t;
        anew(t0, row, t);
        xq = load_codes(a.x + row, t, L);
        if (a.dt_q) {
            raw[0] = load_codes(a.dt_q + row, t, L);
            // What a branch leaves undefined lives on from the tile before, through the loop over states.  (The forms that have these 12
            // registers to spare, and <32, 256, 8>, which keeps 2 others in scratch memory from tile to tile instead, are 0 to 2 % faster
            // as the compiler shares registers out then.)
            if (HALVES) raw[1] = raw[2] = raw[3] = (u32x4)(0u);
        } else if (t + kE <= L) {
#pragma unroll
            for (int q = 0; q < 4; ++q)  // plain, not non-temporal: four loads share a sector
                raw[q] = reinterpret_cast<const u32x4_f *>(a.dt + row + t)[q];
        } else {
#pragma unroll
            for (int i = 0; i < kE; ++i)
                raw[i >> 2][i & 3] = __builtin_bit_cast(uint32_t, a.dt[row + min(t + i, L - 1)]);
        }
    };
    auto stage_bc = [&](const u32x4 &v, int r) {
        f32x4 *dst = (r < NS ? s_B : s_C) + (r & (NS - 1)) * 4 * kLanes + stage_lane;
        const float f = r < NS ? 1.0f : sC;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            dst[q * kLanes] = (f32x4){byte_to_float(v[q], 0) * f, byte_to_float(v[q], 1) * f, byte_to_float(v[q], 2) * f,
                                   byte_to_float(v[q], 3) * f};
    };
    // The lane's 16 codes of every row of B and C that it stages, requested together (one after the other: 6400 channels of two
    // sequences, 4096 tokens 222.8 -> 217.2 us, 5120 channels of one with side inputs 104.7 -> 103.1).
    constexpr int kTrips = (2 * NS + kStagers - 1) / kStagers;
    u32x4 xq, raw[4], bc[kTrips];
    auto load_rows = [&](int t0, int n0) {
#pragma unroll
        for (int i = 0; i < kTrips; ++i) {
            const int r = min(stager + i * kStagers, 2 * NS - 1);
            bc[i] = load_codes((r < NS ? a.B : a.C) + ((size_t)b * N + n0 + (r & (NS - 1))) * L, t0 + kE * stage_lane, L);
        }
    };
    // Where a unit has one workgroup of 2 waves per SIMD, nothing covers the loads between two tiles: there the next tile's are in
    // flight during the loop over states (1536 channels of one sequence, 4096 tokens 44.4 -> 40.9 us, 2048 22.9 -> 21.9).  24
    // channels with 3 waves per SIMD gain 0 to 2 % at 4096 tokens and lose 2.5 % at 1003.
    auto load_ahead = [&](int t0) {
        load_tile(t0, xq, raw);
        load_rows(t0, 0);
    };
    if constexpr (kAlone) load_ahead(0);
    for (int t0 = 0, slot = 0; t0 < L; t0 += kTile, slot = kTiles > 1 ? (slot + 1) % kTiles : 0) {
        if constexpr (!kAlone) load_tile(t0, xq, raw);
        size_t row;
        int t;
        anew(t0, row, t);
        float dt[kE];
        if (a.dt_q) {  // step size = softplus(s_dt code + bias[d]) (Section 3.2)
            const float bias = a.dt_bias ? a.dt_bias[dd] : 0.0f;
#pragma unroll
            for (int i = 0; i < kE; ++i)
                dt[i] = softplus_fast(fmaf(a.dt_scale, byte_to_float(raw[0][i >> 2], i & 3), bias));
        } else {
#pragma unroll
            for (int i = 0; i < kE; ++i) dt[i] = from_bits(raw[i >> 2][i & 3]);
        }
        if (t + kE > L) {  // tokens past the end are identity steps: decay 1, input 0
#pragma unroll
            for (int i = 0; i < kE; ++i) dt[i] = t + i < L ? dt[i] : 0.0f;
        }
        const int last = kTwo && t0 + kScan * kE >= L ? kScan - 1 : LPC - 1;  // the lane that ends the tile
        float u[kE], y[kE];
        float dtsum = 0.0f;
#pragma unroll
        for (int i = 0; i < kE; ++i) {
            const float xf = byte_to_float(xq[i >> 2], i & 3);
            u[i] = dt[i] * (sxB * xf);  // Delta_t x_t with B's scale folded in
            y[i] = Dx * xf;
            dtsum += dt[i];
        }
#pragma unroll 1
        for (int n0 = 0; n0 < N; n0 += NS) {
            if (kTiles == 1 || slot == 0) {
                if (!kAlone) load_rows(t0, n0);
                __syncthreads();  // the workgroup is done with the states before
                // the tile's NS rows each of B and C codes, 16 codes per thread and trip
#pragma unroll
                for (int i = 0; i < kTrips; ++i)
                    if (stager + i * kStagers < 2 * NS) stage_bc(bc[i], stager + i * kStagers);
                if constexpr (kAlone)
                    if (t0 + kTile < L) load_ahead(t0 + kTile);
                __syncthreads();
            } else {  // the states that the wave's lanes have left in front of this tile
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
#pragma unroll 1
            for (int n = 0; n < NS; ++n) {
                const float2 ah = s_AH[ch * N + n0 + n];
                float dec[kE], in[kE];
                float h = 0.0f, P = dtsum * ah.x;
#pragma unroll
                for (int i = 0; i < kE; ++i) dec[i] = dt[i] * ah.x;
                // 64 lanes per channel with all 16 states staged leave 2 waves on a SIMD, 24 channels of 32 lanes 3: too few to
                // cover the LDS reads, and registers to spare.  There the operands are read while the exponentials and the lane scan
                // run (1536 channels of one sequence, 4096 tokens 48.7 -> 45.5 us, 700 tokens 13.7 -> 13.0; 20 channels of 32 lanes
                // on a unit 99.3 -> 95.1).  With 4 waves that changes nothing (306 / 305 us at 4 x 4096 tokens of 5120
                // channels) or spills.
                f32x4 Bn[4], Cn[4];
                auto ahead = [&](f32x4 (&v)[4], const f32x4 *from) {
                    if constexpr (kAhead) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = from[(n * 4 + q) * kLanes + slot * LPC + sub];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                ahead(Bn, s_B);
                exp2_burst(dec, P);  // P becomes the product of the lane's 16 decay factors
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 Bv = kAhead ? Bn[q] : s_B[(n * 4 + q) * kLanes + slot * LPC + sub];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = 4 * q + k;
                        in[i] = u[i] * Bv[k];
                        h = fmaf(dec[i], h, in[i]);
                    }
                }
                ahead(Cn, s_C);
                wave_scan<kScan>(P, h);
                // the state behind this lane's tokens, the pairs up to it applied to the carried state, is the state in
                // front of the next lane's; behind the last lane's it is the state after the tile
                float end = fmaf(P, ah.y, h), from = ah.y;
                if (kTwo) {
                    const float first_end = lane_value(end, kScan - 1);  // (in all lanes' code: the others' `end` has to be there)
                    from = sub < kScan ? ah.y : first_end;
                    end = fmaf(P, from, h);
                }
                float hh = dpp_fetch<0x138, 0xf>(ah.y, end);  // wave_shr:1
                if (LPC < 64 && sub == 0) hh = ah.y;
                float carry = end;
                if (!scan_is_finite(end)) {
                    const bool walked = !HALVES || !group_is_finite<kScan>(end);
                    const float front = walk_lanes<kScan>(ah.y, dec, in);
                    float behind = front;
#pragma unroll
                    for (int i = 0; i < kE; ++i) behind = fmaf(dec[i], behind, in[i]);
                    hh = walked ? front : hh;
                    carry = walked ? behind : carry;
                    if (kTwo) {  // the second tile of 32 lanes goes on from where the first one really ends
                        from = lane_value(carry, kScan - 1);
                        end = fmaf(P, from, h);
                        const bool walk_on = sub >= kScan && !group_is_finite<kScan>(end);
                        const float before = dpp_fetch<0x138, 0xf>(from, end), on = walk_lanes<kScan>(from, dec, in);
                        behind = on;
#pragma unroll
                        for (int i = 0; i < kE; ++i) behind = fmaf(dec[i], behind, in[i]);
                        if (sub >= kScan) {
                            hh = walk_on ? on : sub == kScan ? from : before;
                            carry = walk_on ? behind : end;
                        }
                    }
                }
                if (sub == last) s_AH[ch * N + n0 + n].y = carry;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 Cv = kAhead ? Cn[q] : s_C[(n * 4 + q) * kLanes + slot * LPC + sub];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = 4 * q + k;
                        hh = fmaf(dec[i], hh, in[i]);
                        y[i] = fmaf(Cv[k], hh, y[i]);
                    }
                }
            }
        }
        anew(t0, row, t);
        if (own && t < L) {
            if (a.z) {  // y * SiLU(z) on the gate codes of the lane's 16 tokens (Section 3.2), from the table
                const u32x4 zq = load_codes(a.z + row, t, L);
#pragma unroll
                for (int i = 0; i < kE; ++i) y[i] *= s_silu[(zq[i >> 2] >> (8 * (i & 3))) & 255u];
            }
            uint16_t *yp = a.y + row + t;
            if (t + kE <= L) {
                u32x4 o[2];
#pragma unroll
                for (int i = 0; i < kE; i += 2)
                    o[i >> 3][(i >> 1) & 3] = (uint32_t)f32_to_f16_bits(y[i]) | ((uint32_t)f32_to_f16_bits(y[i + 1]) << 16);
                __builtin_nontemporal_store(o[0], reinterpret_cast<u32x4_h *>(yp));
                __builtin_nontemporal_store(o[1], reinterpret_cast<u32x4_h *>(yp) + 1);
            } else {
#pragma unroll
                for (int i = 0; i < kE; ++i)
                    if (t + i < L) yp[i] = f32_to_f16_bits(y[i]);
            }
        }
    }
    if (fin) {
        __syncthreads();
        for (int i = threadIdx.x; i < kCh * N; i += kThreads) {
            const int c = blk * kCh + i / N;
            if (c < D) fin[((size_t)b * D + c) * N + i % N] = s_AH[i].y;
        }
    }
}

// grid = (channels / (kThreads / LPC), batch)
template <int LPC, int kThreads, int NS>
__global__ __launch_bounds__(kThreads, kThreads == 768 ? 3 : 4) void mamba1_scan_kernel(SsdArgs a, const float *A, const float *init, float *fin)
{
    // separate arrays, so that the compiler sees that the state's write does not touch the C read behind it
    __shared__ f32x4 s_B[NS * 4 * LPC], s_C[NS * 4 * LPC];
    __shared__ float2 s_AH[kThreads / LPC * 16];
    __shared__ float s_silu[256];
    scan_channels<LPC, kThreads, NS>(a, A, init, fin, blockIdx.y, blockIdx.x, s_B, s_C, s_AH, s_silu);
}

// 20 channels per workgroup of 12 waves, one to a compute unit: 16 on 32 lanes each in waves 0..7, the other 4 on 64 lanes each in
// waves 8..11, so that each of the four SIMDs has the work of 5 channels.  (Groups of 32 lanes alone are 6 channels on some or all of
// them: 24 channels per workgroup leave a sixth of the units without one, 20 on 10 waves load two SIMDs with three waves.)  B
// and C of 1024 tokens are staged at a time, one tile of a channel on 64 lanes, two of one on 32.  Bound by the vector ALU as
// above.  5120 channels of one sequence, 24 channels per workgroup / these: 1003 tokens 30.4 / 27.4 us, with state and side inputs
// 32.4 / 29.2, 1500 43.3 / 40.2, 4096 97.8 / 83.6; 3 x 1536 channels, 4096 tokens 94.6 / 80.0.  500 tokens 18.1 / 18.6: half of the
// 64 lanes' tile is empty there.
__global__ __launch_bounds__(768, 3) void mamba1_scan_mixed_kernel(SsdArgs a, const float *A, const float *init, float *fin)
{
    __shared__ f32x4 s_B[16 * 4 * 64], s_C[16 * 4 * 64];
    __shared__ float2 s_AH[20 * 16];
    __shared__ float s_silu[256];
    if (threadIdx.x < 512)
        scan_channels<32, 768, 16, false, 2, true>(a, A, init, fin, blockIdx.y, blockIdx.x, s_B, s_C, s_AH, s_silu);
    else
        scan_channels<64, 768, 16, false, 1, true>(a, A, init, fin, blockIdx.y, blockIdx.x, s_B, s_C, s_AH, s_silu);
}

// The same for groups of 16 channels of all sequences: the first `whole` as workgroups with 32 lanes per channel, each of the others
// as two workgroups with 64 lanes per channel, 8 channels each, 8 states staged at a time, which is the same LDS.  A launch whose
// last round leaves compute units half empty is as slow there as one wave's instruction stream (80 us for 16 channels and 4096
// tokens on a unit, 117 for 32 channels on it); half the channels on twice the waves take 65 us, 41 where a unit has one such half
// (a wave's tile spans 1024 tokens of one channel instead of 512 of two; B and C are converted for 8 channels instead of 16,
// which costs a full chip 5 to 10 %).  Bound as above.  5120 channels of two sequences, 4096 tokens 188 -> 149 us, 1003 tokens 58.4 ->
// 51.7; 1536 channels of two 89 -> 69 and 23.3 -> 20.7.
__global__ __launch_bounds__(512, 4) void mamba1_scan_halves_kernel(SsdArgs a, const float *A, const float *init,
                                                                   float *fin, int whole)
{
    __shared__ f32x4 s_B[16 * 4 * 32], s_C[16 * 4 * 32];  // or of 8 states and 64 lanes
    __shared__ float2 s_AH[16 * 16];
    __shared__ float s_silu[256];
    const int groups = (a.s.headdim + 15) / 16;  // of a sequence
    const int w = blockIdx.x, g = w < whole ? w : whole + (w - whole) / 2;
    const int b = g / groups, c = g - b * groups, half = (w - whole) & 1;
    if (w < whole)
        scan_channels<32, 512, 16, true>(a, A, init, fin, b, c, s_B, s_C, s_AH, s_silu);
    else if (16 * c + 8 * half < a.s.headdim)
        scan_channels<64, 512, 8, true>(a, A, init, fin, b, 2 * c + half, s_B, s_C, s_AH, s_silu);
}

// Any d_state <= 64 and any seqlen: one thread per (sequence, channel), token by token.
constexpr int kMaxStates = 64;
__global__ __launch_bounds__(64) void mamba1_scan_any_kernel(SsdArgs a, const float *A, const float *init, float *fin)
{
    const int D = a.s.headdim, L = a.s.seqlen, N = a.s.d_state;
    const int d = blockIdx.x * 64 + threadIdx.x, b = blockIdx.y;
    if (d >= D) return;
    float h[kMaxStates], A2[kMaxStates];
    for (int n = 0; n < N; ++n) {
        h[n] = init ? init[((size_t)b * D + d) * N + n] : 0.0f;
        A2[n] = A[(size_t)d * N + n] * kLog2e;
    }
    const float sx = x_scale_lookup(a, 0, d), sB = a.B_scales[0], sC = a.C_scales[0];
    const float Dk = a.D ? a.D[d] : 0.0f;
    for (int t = 0; t < L; ++t) {
        const size_t row = ((size_t)b * D + d) * L + t;
        const float dt = step_size(a, row, d), xv = sx * (float)a.x[row];
        const float u = dt * xv * sB;
        float y = 0.0f;
        for (int n = 0; n < N; ++n) {
            const size_t bc = ((size_t)b * N + n) * L + t;
            h[n] = fmaf(__builtin_amdgcn_exp2f(dt * A2[n]), h[n], u * (float)a.B[bc]);
            y = fmaf((float)a.C[bc], h[n], y);
        }
        const float gate = a.z ? silu_of_code(a.z_scale, a.z[row]) : 1.0f;
        a.y[row] = f32_to_f16_bits(fmaf(Dk, xv, sC * y) * gate);
    }
    if (fin)
        for (int n = 0; n < N; ++n) fin[((size_t)b * D + d) * N + n] = h[n];
}

// One generation step on the fp32 state [b, D, N], in place.  N = 16: four lanes share a (sequence, channel) row,
// each moves 16 contiguous bytes of it (consecutive lanes, consecutive addresses), and the four partial sums of y meet
// by data-parallel-primitive moves inside the quad.
__global__ __launch_bounds__(256) void mamba1_decode16_kernel(SsdArgs a, const float *A)
{
    constexpr int kSeq = kDecodeSeqs;  // sequences per thread and trip: the loads of a trip are in flight together
    const int D = a.s.headdim, nb = a.s.batch;
    const int q = blockIdx.x * 256 + threadIdx.x;  // (channel, quarter of its 16 states)
    const int j = q & 3;
    const bool live = (q >> 2) < D;
    const int d = live ? q >> 2 : D - 1;  // lanes past the end redo the last channel and store nothing
    // per channel, once for all sequences of the thread: scale, skip coefficient, the quarter's row of A
    // the cell first: the batch hides the round trip, and the loads of every range's scale cost 1 % of the stream
    const float sx = a.x_scales[cell_lookup(a, 0, d)];
    const float sxB = sx * a.B_scales[0], sC = a.C_scales[0];
    const float Dx = (a.D ? a.D[d] : 0.0f) * sx;
    const f32x4 A2 = *(reinterpret_cast<const f32x4 *>(A + (size_t)d * 16) + j) * kLog2e;
    for (int b0 = blockIdx.y * kSeq; b0 < nb; b0 += gridDim.y * kSeq) {
        f32x4 h[kSeq];
        float dt[kSeq], xc[kSeq];
        uint32_t bq[kSeq], cq[kSeq];
#pragma unroll
        for (int s = 0; s < kSeq; ++s) {
            const int b = min(b0 + s, nb - 1);  // sequences past the end redo the last one and store nothing
            const size_t idx = (size_t)b * D + d;
            h[s] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(a.state + idx * 16) + j);
            dt[s] = step_size(a, idx, d);
            xc[s] = (float)a.x[idx];
            bq[s] = *reinterpret_cast<const uint32_t *>(a.B + (size_t)b * 16 + 4 * j);
            cq[s] = *reinterpret_cast<const uint32_t *>(a.C + (size_t)b * 16 + 4 * j);
        }
#pragma unroll
        for (int s = 0; s < kSeq; ++s) {
            const bool store = live && b0 + s < nb;
            const size_t idx = (size_t)min(b0 + s, nb - 1) * D + d;
            const float u = dt[s] * (sxB * xc[s]);
            float y = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                h[s][k] = fmaf(__builtin_amdgcn_exp2f(dt[s] * A2[k]), h[s][k], u * byte_to_float(bq[s], k));
                y = fmaf(byte_to_float(cq[s], k), h[s][k], y);
            }
            if (store) __builtin_nontemporal_store(h[s], reinterpret_cast<f32x4 *>(a.state + idx * 16) + j);
            y = group_sum<4>(y);
            if (j == 0 && store) {
                const float gate = a.z ? silu_of_code(a.z_scale, a.z[idx]) : 1.0f;
                a.y[idx] = f32_to_f16_bits(fmaf(Dx, xc[s], sC * y) * gate);
            }
        }
    }
}

// Any d_state: one thread per (sequence, channel).
__global__ __launch_bounds__(256) void mamba1_decode_any_kernel(SsdArgs a, const float *A)
{
    const int D = a.s.headdim, N = a.s.d_state;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)a.s.batch * D) return;
    const int b = (int)(idx / D), d = (int)(idx - (size_t)b * D);
    const float dt = step_size(a, idx, d), xv = x_scale_lookup(a, 0, d) * (float)a.x[idx];
    const float u = dt * xv * a.B_scales[0];
    float *st = a.state + idx * N;
    const float *Ar = A + (size_t)d * N;
    const int8_t *Bq = a.B + (size_t)b * N, *Cq = a.C + (size_t)b * N;
    float y = 0.0f;
    for (int n = 0; n < N; ++n) {
        const float hn = fmaf(__builtin_amdgcn_exp2f(dt * Ar[n] * kLog2e), st[n], u * (float)Bq[n]);
        st[n] = hn;
        y = fmaf((float)Cq[n], hn, y);
    }
    const float gate = a.z ? silu_of_code(a.z_scale, a.z[idx]) : 1.0f;
    a.y[idx] = f32_to_f16_bits(fmaf(a.D ? a.D[d] : 0.0f, xv, a.C_scales[0] * y) * gate);
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

template <int LPC, int kThreads, int NS>
hipError_t launch_scan(const SsdArgs &a, const float *A, const float *init, float *fin, hipStream_t stream)
{
    constexpr int channels = kThreads / LPC;  // of a workgroup
    const dim3 grid((unsigned)((a.s.headdim + channels - 1) / channels), (unsigned)a.s.batch);
    hipLaunchKernelGGL((mamba1_scan_kernel<LPC, kThreads, NS>), grid, dim3(kThreads), 0, stream, a, A, init, fin);
    return hipGetLastError();
}

// Groups of 16 channels in the full rounds of two per compute unit.
int64_t whole_groups(const quamba_ssd_shape_t &s)
{
    const int64_t round = 2 * (int64_t)compute_units();
    return (int64_t)s.batch * ((s.headdim + 15) / 16) / round * round;
}

}  // namespace

bool mamba1_scan_supports_any(const quamba_ssd_shape_t &s) { return s.d_state <= kMaxStates; }

Mamba1Form mamba1_scan_form(const quamba_ssd_shape_t &s)
{
    const int D = s.headdim, cus = compute_units();
    const int64_t batch = s.batch, L = s.seqlen;
    if ((s.flags & QUAMBA_FLAG_GENERIC_KERNEL) || s.d_state != 16 || L < kE) return Mamba1Form::any;
    // Lanes per channel: 16 for sequences one such tile (256 tokens) holds, where more lanes would idle; 64 when there
    // are so few channels that a workgroup per compute unit is all there is, which halves the tiles each walks.
    if (L <= 16 * kE) return Mamba1Form::lanes16;
    auto per_cu = [&](int ch) { return (batch * ((D + ch - 1) / ch) + cus - 1) / cus * ch; };
    if (L > 32 * kE && per_cu(8) <= 8) return Mamba1Form::lanes64;
    // Else the time follows the channels of the fullest compute unit times the tokens of their tiles (about 1 us per
    // 1000, from 1003 tokens up).  16 channels of 32 lanes in a workgroup; 8 where that spreads the channels more evenly
    // (6400 channels, two sequences: 56 instead of 64 on a unit; 16 / 8 channels 1003 tokens 64.2 / 62.0 us, 4096 224.5 / 210.5; where
    // it does not, its staging costs up to 5 %: 4 x 1003 tokens of 5120 channels 82 against 84 us); 32 of 16 lanes where their
    // tiles of 256 tokens leave less over (3 x 700 tokens of 5120 channels 63.5 -> 47.7 us).  A difference below an
    // eighth does not pay.
    auto cost = [&](int ch, int tile) { return per_cu(ch) * ((L + tile - 1) / tile * tile); };
    const int64_t c16 = cost(16, 32 * kE), c8 = cost(8, 32 * kE), c32 = cost(32, 16 * kE);
    // Halves of groups of 16 channels behind the rounds of two groups per compute unit, where a unit has at most one group of
    // the rest.  Costs in channels of a full unit times tokens: the rest takes 22 (one group on a unit) as whole groups, 18 as
    // halves, 13 where a unit has one half; but a half's tiles are twice as long, so that it walks more padded tokens (9 : 10
    // and 6 : 10 per tile of 1024 against 512; 1500 tokens of 192 groups 36.1 / 36.5 us, of 512 + 128 groups 77 -> 68).  Behind
    // two rounds and more (1280 groups 308 / 309 us) a group per unit starts as units come free and gains nothing any more; at
    // most a half per unit does until about eight rounds (2112 groups 409 -> 380 us, 4160 groups 979 -> 968).
    const int64_t groups = batch * ((D + 15) / 16), whole = whole_groups(s), rest = groups - whole;
    const int64_t tiles = (L + 32 * kE - 1) / (32 * kE), long_tiles = (tiles + 1) / 2;
    const bool few = 2 * rest <= cus;
    // groups of 8 channels in workgroups of 256 threads, in the same measure: four on a unit 32, three 29, two 24, one 22
    const int64_t eights = per_cu(8) / 8, alone[4] = {0, 22, 24, 29}, tokens = tiles * 32 * kE;
    const int64_t halves = 16 * (whole / cus) * tokens + (few ? 13 : 18) * long_tiles * 64 * kE;
    if (rest > 0 && rest <= cus && whole <= (few ? 16 : 2) * cus && (few ? 6 : 9) * long_tiles <= 5 * tiles && halves <= c32 &&
        halves <= (eights / 4 * 32 + alone[eights % 4]) * tokens)
        return Mamba1Form::halves;
    // 24 channels in one workgroup per compute unit where they hold all channels and groups of 16 do not: 4 x 1536 channels, 4096
    // tokens 110.6 -> 104.1 us, 1003 tokens with side inputs 35.5 -> 31.5; 5120 channels of one sequence 104.2 -> 92.5
    // (those were three and two workgroups of 8 channels per unit).  Where 20 per unit hold all channels: mamba1_scan_mixes.
    if (groups > cus && eights > 2 && batch * ((D + 23) / 24) <= cus) return Mamba1Form::channels24;
    if (9 * std::min(c8, c32) <= 8 * c16) return c8 <= c32 ? Mamba1Form::channels8 : Mamba1Form::lanes16;
    return Mamba1Form::lanes32;
}

// The one workgroup per unit of Mamba1Form::channels24 takes 20 channels, some on 64 lanes, where these hold all and the sequences
// are longer than a tile of 32 lanes (measured at mamba1_scan_mixed_kernel).
bool mamba1_scan_mixes(const quamba_ssd_shape_t &s)
{
    return mamba1_scan_form(s) == Mamba1Form::channels24 && s.seqlen > 32 * kE &&
           (int64_t)s.batch * ((s.headdim + 19) / 20) <= compute_units();
}

hipError_t launch_mamba1_scan(const SsdArgs &a, const float *A, const float *init, float *fin, hipStream_t stream)
{
    switch (mamba1_scan_form(a.s)) {
        case Mamba1Form::lanes16: return launch_scan<16, 512, 16>(a, A, init, fin, stream);
        case Mamba1Form::lanes32: return launch_scan<32, 512, 16>(a, A, init, fin, stream);
        case Mamba1Form::lanes64: return launch_scan<64, 512, 16>(a, A, init, fin, stream);
        case Mamba1Form::channels8: return launch_scan<32, 256, 8>(a, A, init, fin, stream);
        case Mamba1Form::channels24:
            if (!mamba1_scan_mixes(a.s)) return launch_scan<32, 768, 16>(a, A, init, fin, stream);
            hipLaunchKernelGGL(mamba1_scan_mixed_kernel, dim3((unsigned)((a.s.headdim + 19) / 20), (unsigned)a.s.batch), dim3(768), 0, stream, a,
                               A, init, fin);
            return hipGetLastError();
        case Mamba1Form::halves: {
            const int64_t groups = (int64_t)a.s.batch * ((a.s.headdim + 15) / 16), whole = whole_groups(a.s);
            hipLaunchKernelGGL(mamba1_scan_halves_kernel, dim3((unsigned)(whole + 2 * (groups - whole))), dim3(512), 0, stream, a, A,
                               init, fin, (int)whole);
            return hipGetLastError();
        }
        default: break;
    }
    const dim3 grid((unsigned)((a.s.headdim + 63) / 64), (unsigned)a.s.batch);
    hipLaunchKernelGGL(mamba1_scan_any_kernel, grid, dim3(64), 0, stream, a, A, init, fin);
    return hipGetLastError();
}

hipError_t launch_mamba1_decode(const SsdArgs &a, const float *A, hipStream_t stream)
{
    const size_t total = (size_t)a.s.batch * a.s.headdim;
    if (a.s.d_state == 16 && aligned16(a.state) && aligned16(A) && reinterpret_cast<uintptr_t>(a.B) % 4 == 0 &&
        reinterpret_cast<uintptr_t>(a.C) % 4 == 0) {
        // x: the (channel, quarter) pairs; y: groups of kDecodeSeqs sequences (a thread loops if the batch has more
        // groups than the grid's y dimension may hold)
        const dim3 grid((unsigned)((4 * (size_t)a.s.headdim + 255) / 256),
                        (unsigned)std::min((a.s.batch + kDecodeSeqs - 1) / kDecodeSeqs, 65535));
        hipLaunchKernelGGL(mamba1_decode16_kernel, grid, dim3(256), 0, stream, a, A);
    } else {
        hipLaunchKernelGGL(mamba1_decode_any_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, a, A);
    }
    return hipGetLastError();
}

}  // namespace quamba
