// Chunked prefill of batches of at most one (sequence, head) pair per compute unit, where every pair (with half a pair per
// unit: every channel half of every pair, or every half or whole head of every segment of its sequence) has a unit to itself; and of
// up to one and a third, whose units share the pairs (shared_rounds in prefill_mfma.hip).
//
// The arithmetic is that of prefill_mfma_kernel (prefill_mfma.hip describes it), for 32 (PT = 1) or all 64 (PT = 2) of a head's
// channels.  What bounds such a launch is the serial walk over the chunks: a lone wave issues an instruction every 4
// cycles and waits alone for each result, and with 8 waves in two phases between two barriers a chunk of 32 channels took 2.7 us.  Here a workgroup has 16 waves, four
// to a SIMD, in four roles that work side by side on everything a chunk needs, and one barrier per chunk:
//   waves  0..3   the later terms of a 32-token block's outputs (the pair in front of the diagonal of the two longer blocks,
//                 the diagonal, the skip term) and, one chunk later, its scaled outputs
//   waves  4..7   the earlier terms (carried state, first block pairs), left in LDS for the wave that writes the outputs;
//                 the one of block 0, which has no pairs, also forms the next chunk's token weights
//   waves  8..11  the state update (a quarter of the states each), and the state as fp16 for the next chunk
//   waves 12..15  staging of the next chunk: x, gate codes, B and C rows
// so that LDS holds two of what a chunk reads (up to the whole 160 KB, which one workgroup per unit may take).  C rows come
// through LDS: loaded by the lanes that use them, 16 bytes a lane and row, they kept the address unit busy for 2000 cycles of
// a chunk.  The skip term is a product of the x codes with a diagonal matrix (its fp16 coefficient and the remainder), the causal
// mask an AND on the narrowed scores, and the carried state's decay factor is applied to the finished sums: fewer vector
// instructions than selects and scaled operands, and fewer roundings (error of y against 64 bits 2.5 to 3.0e-4, 8-wave kernel
// 2.6 to 3.2e-4).
//
// Segments of a sequence are walked by workgroups of a few chunks, whose start counts: there the waves stand the other way round, in
// the order in which the first chunk needs them.  The last of 16 waves starts 2200 cycles after the first, and with the staging waves
// last the first chunk was staged at 5900 to 7900 cycles, now at 4500 to 6000 (24 heads of 2048 tokens in 4 segments of halves 24.4 ->
// 23.5 us).  A SIMD serves its oldest wave first, and a chunk takes longer when that is a staging wave (64 channels 4700 cycles
// instead of 4000), so priorities restore the other order of service.  They cost a chunk 1 %: 12 chunks of 128 heads with gate and
// step-size codes 45.8 -> 46.3 us, so unsplit calls do without both.
//
// Measured with the final state (the best of the 8-wave kernel's launches, whole, cut into segments or in channel halves /
// this kernel): 128 heads, one sequence of 1531 tokens with gate and step-size codes 49.4 / 34.9 us, 2500 tokens 56 / 46; 120
// pairs, 1000 tokens 32.2 / 22.0; 80 heads, 1000 tokens 27.4 / 20.8; 24 heads, 2048 tokens (8 segments of whole heads) 24.3 / 19.8,
// 500 tokens 14.3 / 11.9; 40 heads, 2048 tokens (6 segments of whole heads) 29.5 / 26.1; two sequences of 128 heads, 1024 tokens 36.1 /
// 30.6, 4096 tokens 128 / 107, 1531 tokens with gate and codes 64.4 / 47.5.  By cycle counters read in the kernel (a build of its
// own) a chunk of 32 channels takes 4000 cycles, 4600 with the
// two-term state update; the roles' waves wait 500 to 1500 of them at the barrier, the vector ALUs issue 3000 (the hardware's
// counters, profiles/short_prompts_and_mixed_hadamard.txt, have 840 instructions per SIMD and chunk, the launch's set-up
// included, 960 with gate and step-size codes).  A chunk of 64 channels takes 5600 (6200): its state waves are busy for 5100 of
// them, the others for 3600 to 4600, and LDS for 3000.  Wave priorities for the state waves cost 1 to 3 %, their operands requested
// two or three steps ahead change nothing.  Two rounds of this kernel are slower than two workgroups of 8 waves side by side
// (512 pairs, 4096 tokens: 193 / 169 us; 384 pairs, 2048 tokens 105 / 89, with the units sharing the pairs 86).
#include "prefill_tiles.h"

namespace quamba {
namespace {

constexpr int kWideThreads = 1024;

// LDS map (bytes) for PT 32-channel tiles per workgroup: two sets of what a chunk reads.  With 64 channels two sets of everything
// would not fit: the state, the early terms and, with a gate, the C rows then have one place, and who writes it waits until
// its readers have said that they are done with the chunk before (counters behind the tables).
template <int PT, bool GATED>
struct WideLds {
    static constexpr bool kOneH = PT == 2, kOnePart = PT == 2, kOneC = PT == 2 && GATED;
    static constexpr int kPw = 32 * PT;                         // channels of the workgroup
    static constexpr int kXsStride = PT == 2 ? 64 : 48;         // halves per row of x [token][p]
    static constexpr int kZsStride = kPw + 8;                   // bytes per row of gate codes [token][p]
    static constexpr int kC = kQ * kN, kH = 2 * kPw * kHsStride, kPart = kNBlk * PT * 4 * 64 * 16;
    static constexpr int kOffCum = 0;                           // float[128]
    static constexpr int kOffLoc = kOffCum + 4 * kQ;            // float[128]
    static constexpr int kOffDt = kOffLoc + 4 * kQ;             // float[128]
    static constexpr int kOffW2 = kOffDt + 4 * kQ;              // float[128]
    static constexpr int kOffWe = kOffW2 + 4 * kQ;              // fp16[128]
    static constexpr int kOffWs = kOffWe + 2 * kQ;              // fp16[128]
    static constexpr int kOffWd = kOffWs + 2 * kQ;              // fp16[128]
    static constexpr int kOffTot = kOffWd + 2 * kQ;             // float[4]
    static constexpr int kOffGap = kOffTot + 4 * kNBlk;         // float[4][4]
    static constexpr int kOffBq = kOffGap + 4 * kNBlk * kNBlk;  // int8 [128][144]
    static constexpr int kOffXs = kOffBq + kQ * kBqStride;      // fp16 [128][kXsStride]
    static constexpr int kOffZs = kOffXs + 2 * kQ * kXsStride;  // int8 [128][kZsStride]
    static constexpr int kSet = kOffZs + (GATED ? kQ * kZsStride : 0);
    static constexpr int kOffCq = 2 * kSet;                     // int8 [128][128], 16-byte pieces of row r at piece ^ (r & 7)
    static constexpr int kOffHs = kOffCq + (kOneC ? 1 : 2) * kC;        // fp16 [kPw][136]
    static constexpr int kOffPart = kOffHs + (kOneH ? 1 : 2) * kH;      // float[4 blocks][PT * 4][64 lanes][4]
    static constexpr int kOffSx = kOffPart + (kOnePart ? 1 : 2) * kPart;  // float[kPw]
    static constexpr int kOffDone = kOffSx + 4 * kPw;           // int[16]: chunks read of the early terms [4], the state [4], C [8]
    static constexpr int kOffLeft = kOffDone + 4 * 16;          // int: a piece of shared rounds goes on from the one in front of it
    static constexpr int kOffSilu = kOffLeft + 16;              // float[256]
    static constexpr int kOffKeep = kOffSilu + (GATED ? 4 * 256 : 0);   // uint32[2][64 lanes][4] (PT == 2): the causal mask
    static constexpr int kBytes = kOffKeep + (PT == 2 ? 2048 : 0);
    static_assert(kOffBq % 16 == 0 && kOffHs % 16 == 0 && kOffXs % 16 == 0 && kSet % 16 == 0 && kOffDone % 16 == 0, "16-byte alignment");
    static_assert(kBytes <= (int)kLdsPerCu, "one workgroup per compute unit");
};

// Byte offset of 8 bytes of x in a row of the LDS: 32-byte piece (16 channels), 8-byte part.  Rows of 64 channels have no room for
// padding: their pieces change places with bit 1 of the row, which puts the 4 rows x 32 bytes that the lane groups of a
// transposing read fetch together on distinct banks.
template <int PT>
__device__ __forceinline__ int x_part(int row, int piece, int part)
{
    return (PT == 2 ? piece ^ (row & 2) : piece) * 32 + part * 8;
}

template <bool PRECISE, int PT, bool GATED, Walk WALK>
__global__ __launch_bounds__(kWideThreads, 4) void prefill_wide_kernel(typename WalkArgs<WALK>::type a)
{
    constexpr bool SEG = WALK == Walk::segment, SHARED = WALK == Walk::shared;
    static_assert(!SHARED || PT == 2, "pieces are of whole heads");
    typedef WideLds<PT, GATED> LY;
    constexpr int kPw = LY::kPw, kXsStride = LY::kXsStride, kZsStride = LY::kZsStride;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int *s_done = reinterpret_cast<int *>(smem + LY::kOffDone);
    auto c_rows = [&](int buf) { return smem + LY::kOffCq + (LY::kOneC ? 0 : buf * LY::kC); };
    auto h_rows = [&](int buf) { return smem + LY::kOffHs + (LY::kOneH ? 0 : buf * LY::kH); };
    auto part_of = [&](int buf) { return reinterpret_cast<f32x4 *>(smem + LY::kOffPart + (LY::kOnePart ? 0 : buf * LY::kPart)); };
    // "Chunks 0 .. n-1 of this walk are read" and the wait for it.  A reader says so in the phase of chunk n-1 or n without
    // waiting for anyone but the readers of the early terms (which wait for nobody), so every wait ends.
    auto done = [&](int slot, int n) { __hip_atomic_store(s_done + slot, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto wait_done = [&](int slot, int n) {
        while (__hip_atomic_load(s_done + slot, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < n) __builtin_amdgcn_s_sleep(1);
    };
    float *s_sx = reinterpret_cast<float *>(smem + LY::kOffSx);
    float *s_silu = reinterpret_cast<float *>(smem + LY::kOffSilu);

    const int L = a.s.seqlen, H = a.s.nheads, G = a.s.ngroups;
    // All of the arguments' lines asked for at once, where the compiler would wait for each before it asks for the next (not where a
    // register would have to go to scratch memory for it).
    if (PT == 1 || SEG)
        asm volatile("" ::"s"(a.x), "s"(a.B), "s"(a.C), "s"(a.A), "s"(a.D), "s"(a.seg_state), "s"(a.inv_heads));
    const int npairs = a.s.batch * H;
    const int seg = SEG ? quotient((int)blockIdx.x, a.inv_wgs_per_seg) : 0;
    const int nchunks = (L + kQ - 1) / kQ;
    int c_begin = SEG ? seg * a.seg_chunks : 0;
    int c_end = (SEG && seg + 1 < a.nseg) ? c_begin + a.seg_chunks : nchunks;
    const int bid = SEG ? (int)blockIdx.x - seg * a.wgs_per_seg : (int)blockIdx.x;
    int pair = bid, half = 0, cut = 0;
    if constexpr (SHARED)
        if (!shared_piece(a, pair, cut, c_begin, c_end)) return;
    bool convert_init = a.init_state && c_begin == 0;  // the caller's initial state stands in front of the first chunk
    if (PT == 1) {
        const int full = npairs >> 3;
        if (bid < 16 * full) {
            pair = (bid & 7) | ((bid >> 4) << 3);
            half = (bid >> 3) & 1;
        } else {
            const int t = bid - 16 * full, r = npairs - 8 * full;
            pair = 8 * full + t % r;
            half = t / r;
        }
    }
    const int p_base = 32 * half;
    int b, h, g;
    place_of(a, pair, b, h, g);
    const int bh = b * H + h;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave16 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = SEG ? 3 - (wave16 >> 2) : wave16 >> 2, wave = wave16 & 3;
    const int tid4 = tid & 255;
    if (tid < 16) s_done[tid] = 0;  // read and written behind the first barrier
    if (SEG) {  // (see the top: the outputs' waves are the youngest of their SIMD)
        if (role == 0) __builtin_amdgcn_s_setprio(3);
        else if (role == 1) __builtin_amdgcn_s_setprio(2);
        else if (role == 2) __builtin_amdgcn_s_setprio(1);
    }
    // Lane-derived values are made anew in every chunk (fresh_lane): kept across the loop over chunks, the addresses formed
    // from them would push other values into scratch memory.
    int l32 = lane & 31, hb = lane >> 5;
    auto new_lane = [&]() {
        const int ln = fresh_lane();
        l32 = ln & 31;
        hb = ln >> 5;
    };

    // A piece that begins behind the first chunk goes on from the state that the piece in front of it leaves, for which the first
    // state wave looks; without it, it starts over (true).
    int *s_left = reinterpret_cast<int *>(smem + LY::kOffLeft);
    auto starts_over = [&]() {
        if (!SHARED || c_begin == 0) return false;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(*s_left)) return false;
        c_begin = 0;
        convert_init = a.init_state != nullptr;
        return true;
    };

    const float Ah = a.A[h] * 1.44269504088896340736f;
    const float Dh = a.D ? a.D[h] : 0.0f;
    const float sB = a.B_scales[g], sC = a.C_scales[g];
    const float y_scale = sB * sC * (1.0f / (kNarrow * kAcc));
    const float d_acc = Dh / (y_scale * kXs);
    const bool d_by_mfma = fabsf(d_acc) < 3.0e4f;
    const float dead = (a.s.flags & QUAMBA_FLAG_NO_DECAY_SKIP) ? __builtin_inff() : kDead;
    typedef uint32_t xvec __attribute__((ext_vector_type(PT)));
    const uint32_t x_row = (uint32_t)H * kP, b_row = (uint32_t)G * kN, dt_row = (uint32_t)H * 4u;

    // The chunk's token weights from its step sizes, two tokens per lane (one wave; the weights are those of
    // prefill_mfma_kernel, from the same sums).
    auto load_dt = [&](int c, float &dt0, float &dt1) {
        const int t0 = c * kQ;
        const int nv = min(kQ, L - t0);
        const size_t tokbase = (size_t)b * L + t0;
        const int ln = 32 * hb + l32;
        const uint32_t r0 = (uint32_t)min(2 * ln, nv - 1), r1 = (uint32_t)min(2 * ln + 1, nv - 1);
        if (a.dt_q) {
            const int8_t *qbase = a.dt_q + tokbase * H + h;
            dt0 = __builtin_bit_cast(float, (int)qbase[r0 * (uint32_t)H]);
            dt1 = __builtin_bit_cast(float, (int)qbase[r1 * (uint32_t)H]);
        } else {
            const char *dbase = reinterpret_cast<const char *>(a.dt + tokbase * H + h);
            dt0 = *reinterpret_cast<const float *>(dbase + r0 * dt_row);
            dt1 = *reinterpret_cast<const float *>(dbase + r1 * dt_row);
        }
    };
    auto token_weights = [&](int c, unsigned char *set, float d0, float d1) {
        const int nv = min(kQ, L - c * kQ);
        const int ln = 32 * hb + l32;
        float *s_cum = reinterpret_cast<float *>(set + LY::kOffCum);
        float *s_loc = reinterpret_cast<float *>(set + LY::kOffLoc);
        float *s_dt = reinterpret_cast<float *>(set + LY::kOffDt);
        float *s_w2 = reinterpret_cast<float *>(set + LY::kOffW2);
        _Float16 *s_we = reinterpret_cast<_Float16 *>(set + LY::kOffWe);
        _Float16 *s_ws = reinterpret_cast<_Float16 *>(set + LY::kOffWs);
        _Float16 *s_wd = reinterpret_cast<_Float16 *>(set + LY::kOffWd);
        float *s_tot = reinterpret_cast<float *>(set + LY::kOffTot);
        float *s_gap = reinterpret_cast<float *>(set + LY::kOffGap);
        if (a.dt_q) {
            const float bias = a.dt_bias ? a.dt_bias[h] : 0.0f;
            const float v0 = a.dt_scale * (float)__builtin_bit_cast(int, d0) + bias;
            const float v1 = a.dt_scale * (float)__builtin_bit_cast(int, d1) + bias;
            d0 = fmaxf(v0, 0.0f) + log1pf(expf(-fabsf(v0)));
            d1 = fmaxf(v1, 0.0f) + log1pf(expf(-fabsf(v1)));
        }
        if (2 * ln >= nv) d0 = 0.0f;
        if (2 * ln + 1 >= nv) d1 = 0.0f;
        const float a0 = d0 * Ah, a1 = d1 * Ah;
        float loc1;
        const float cum1 = wave_inclusive_scan(a0 + a1, loc1), cum0 = cum1 - a1;
        const float loc0 = loc1 - a1;
        const float suf1 = row_suffix_sum_exclusive(a0 + a1), suf0 = suf1 + a1;
        const float q0 = d0 * (kNarrow / kXs), q1 = d1 * (kNarrow / kXs);
        d0 *= kAcc / kXs;
        d1 *= kAcc / kXs;
        const float e0 = exp2_fast(suf0), e1 = exp2_fast(suf1);
        *reinterpret_cast<float2 *>(s_cum + 2 * ln) = make_float2(cum0, cum1);
        *reinterpret_cast<float2 *>(s_loc + 2 * ln) = make_float2(loc0, loc1);
        const float T1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, loc1), 31));
        const float T2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, loc1), 47));
        const float T3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, loc1), 63));
        if ((ln & 15) == 15) s_tot[ln >> 4] = loc1;
        if (ln < kNBlk * kNBlk) s_gap[ln] = ln == 8 ? T1 : ln == 12 ? T1 + T2 : ln == 13 ? T2 : 0.0f;
        *reinterpret_cast<float2 *>(s_dt + 2 * ln) = make_float2(d0 * kNarrow, d1 * kNarrow);
        *reinterpret_cast<float2 *>(s_w2 + 2 * ln) =
            make_float2(exp2_fast(-loc0) * d0 * kNarrow, exp2_fast(-loc1) * d1 * kNarrow);
        const int pos = tok_pos(2 * ln);  // the fp16 weights lie in the order of the x and B rows: 8 of a lane are consecutive
        *reinterpret_cast<f16x2 *>(s_we + pos) = (f16x2){(_Float16)(e0 * d0), (_Float16)(e1 * d1)};
        if (!PRECISE) {
            const int row = ln >> 4;
            const float later = row == 0 ? T1 + (T2 + T3) : row == 1 ? T2 + T3 : row == 2 ? T3 : 0.0f;
            *reinterpret_cast<f16x2 *>(s_ws + pos) = (f16x2){(_Float16)(exp2_fast(suf0 + later) * q0),
                                                                  (_Float16)(exp2_fast(suf1 + later) * q1)};
        } else {
            f16x2 wq, wd;
            const float w[2] = {e0 * q0, e1 * q1};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float q =
                    __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, w[i]) + 0x00080000u) & 0xfff00000u);
                wq[i] = (_Float16)q;
                wd[i] = (_Float16)(q > 0.0f ? (w[i] - q) / q : 0.0f);
            }
            *reinterpret_cast<f16x2 *>(s_ws + pos) = wq;
            *reinterpret_cast<f16x2 *>(s_wd + pos) = wd;
        }
    };

    if (role < 2) {
        // ================= output waves =================
        // B and C rows in registers, int8 score tile G^T of (block sb, the wave's block)
        auto load_c_rows = [&](int buf, int tb, i32x4(&ct)[4]) {
            const unsigned char *row = c_rows(buf) + (tb * kBlk + l32) * kN;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                ct[kk] = *reinterpret_cast<const i32x4 *>(row + 16 * ((2 * kk + hb) ^ (l32 & 7)));
        };
        auto score_tile = [&](const unsigned char *set, int sb, const i32x4(&ct)[4]) {
            const unsigned char *row = set + LY::kOffBq + (sb * kBlk + tok_pos(l32)) * kBqStride + hb * 16;
            i32x4 bq[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) bq[kk] = *reinterpret_cast<const i32x4 *>(row + 32 * kk);
            i32x16 gi;
#pragma unroll
            for (int r = 0; r < 16; ++r) gi[r] = 0;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) gi = __builtin_amdgcn_mfma_i32_32x32x32_i8(bq[kk], ct[kk], gi, 0, 0, 0);
            return gi;
        };
        // x of 16 tokens (first token in the wave's LDS order: row), operand of the products with the score tiles
        auto load_x = [&](const unsigned char *set, int row, int pt) {
            const int i16 = l32 & 15, c16 = l32 >> 4, r = 8 * hb + (i16 >> 2);
            return lds_read_tr16x8<kXsStride>(set + LY::kOffXs + (row + r) * kXsStride * 2 + x_part<PT>(r, 2 * pt + c16, i16 & 3));
        };
        // acc += x^T (G^T exp(cum_t - m) exp(m - cum_s) dt_s) of the block pairs sb0 <= sb < end in front of the diagonal;
        // gi holds the tile of sb0 and, with `more`, ends as the tile of `end`
        auto off_diagonal = [&](const unsigned char *set, int tb, int sb0, int end, bool more, float loc_t,
                                const i32x4(&ct)[4], i32x16 &gi, f32x16 (&acc)[PT]) {
            const float *s_gap = reinterpret_cast<const float *>(set + LY::kOffGap);
            const _Float16 *s_we = reinterpret_cast<const _Float16 *>(set + LY::kOffWe);
            for (int sb = sb0; sb < end; ++sb) {
                if (PT == 2) new_lane();
                f16x8 x0[PT], x1[PT];
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) {
                    x0[pt] = load_x(set, sb * kBlk, pt);
                    x1[pt] = load_x(set, sb * kBlk + 16, pt);
                }
                const f16x8 w0 = *reinterpret_cast<const f16x8 *>(s_we + sb * kBlk + 8 * hb);
                const f16x8 w1 = *reinterpret_cast<const f16x8 *>(s_we + sb * kBlk + 16 + 8 * hb);
                const float rowf = exp2_fast(loc_t + s_gap[tb * kNBlk + sb]) * kNarrow;
                float lv[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) lv[r] = (float)gi[r] * rowf;
                const f16x8 l0 = pack_f16x8(lv) * w0, l1 = pack_f16x8(lv + 8) * w1;
                __builtin_amdgcn_sched_barrier(0);
                if (more || sb + 1 < end) gi = score_tile(set, sb + 1, ct);
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) {
                    acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0[pt], l0, acc[pt], 0, 0, 0);
                    acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[pt], l1, acc[pt], 0, 0, 0);
                }
            }
        };
        // first block in front of the nearest one whose decay towards block tb is alive (the nearest one if none is; between the
        // two lies nothing that could decay)
        auto first_alive = [&](const float *s_cum, int tb, float r_tb) {
            const float m0 = s_cum[kBlk - 1], m1 = s_cum[2 * kBlk - 1];
            return __builtin_amdgcn_readfirstlane((1 < tb && r_tb - m0 < -dead) + (2 < tb && r_tb - m1 < -dead));
        };

        if (role == 0) {
            // ---- the later terms and the outputs of block `wave` ----
            const int tb = wave, mid = tb >= 2 ? tb - 1 : tb;
            if (SEG) new_lane();  // (not kept from in front of the other roles' code)
            if (tid4 < kPw) s_sx[tid4] = x_scale_lookup_wide(a, h, p_base + tid4) * (d_by_mfma ? y_scale : 1.0f);
            if (GATED) s_silu[tid4] = silu_of_code(a.z_scale, (int8_t)tid4);
            // per lane (token t of the block): which of its 16 score rows s are at or in front of t, two to a dword; with 64 channels
            // they wait in LDS, the registers are the sums'
            u32x4 keep[2];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const int s = 8 * (r >> 2) + 4 * hb + (r & 3);
                keep[r >> 3][(r >> 1) & 3] = (s <= l32 ? 0xffffu : 0u) | (s + 1 <= l32 ? 0xffff0000u : 0u);
            }
            u32x4 *s_keep = reinterpret_cast<u32x4 *>(smem + LY::kOffKeep);
            if (PT == 2 && wave < 2) s_keep[64 * wave + lane] = keep[wave];
            // the skip term's coefficient on the diagonal, as fp16 and its remainder, as operands of their own
            const float d_sel = d_by_mfma ? d_acc : 0.0f;
            const uint32_t d16 = f32_to_f16_bits(d_sel);
            const uint32_t d16_rest = f32_to_f16_bits(d_sel - (float)(_Float16)d_sel);
            auto diagonal = [&](uint32_t bits, f16x8(&op)[2]) {
                const bool own = ((l32 >> 2) & 1) == hb;  // row s == t is register 4 (t / 8) + t % 4
                const int at = own ? 2 * (l32 >> 3) + ((l32 >> 1) & 1) : 8;
                const uint32_t val = l32 & 1 ? bits << 16 : bits;
                u32x4 w[2];
#pragma unroll
                for (int k = 0; k < 8; ++k) w[k >> 2][k & 3] = at == k ? val : 0u;
                op[0] = __builtin_bit_cast(f16x8, w[0]);
                op[1] = __builtin_bit_cast(f16x8, w[1]);
            };
            f16x8 skip[2], skip_rest[2];
            if (PT == 1) {
                diagonal(d16, skip);
                diagonal(d16_rest, skip_rest);
            }
            starts_over();
            if (convert_init) __syncthreads();
            __syncthreads();  // the first chunk is staged

            f32x16 acc[PT];
            uint32_t zq[PT][4];
            f16x4 xq[PT][4];
            // outputs of the block's tokens of chunk c, from acc and what the early wave has left in LDS
            auto epilogue = [&](int c, int buf) {
                const int t0 = c * kQ;
                const int nv = min(kQ, L - t0);
                const int tl = tb * kBlk + l32;
                uint16_t *yrow = a.y + ((((size_t)b * L + t0) + min(tl, nv - 1)) * H + h) * kP + p_base + 8 * hb;
                const f32x4 *part = part_of(buf) + tb * PT * 4 * 64 + 32 * hb + l32;
#pragma unroll
                for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const f32x4 v4 = part[(pt * 4 + rg) * 64];
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[pt][4 * rg + i] += v4[i];
                    }
                if (LY::kOnePart) done(tb, c - c_begin + 1);
                if (!d_by_mfma) {
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            acc[pt][r] = fmaf(y_scale, acc[pt][r], Dh * ((float)xq[pt][r >> 2][r & 3] * (1.0f / kXs)));
                }
#pragma unroll
                for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        uint32_t w[2][2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int rg = 2 * j + e;
                            const f32x4 k4 = *reinterpret_cast<const f32x4 *>(s_sx + 32 * pt + 8 * rg + 4 * hb);
                            f16x4 o;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                float v = k4[i] * acc[pt][4 * rg + i];
                                if (GATED) v *= s_silu[(zq[pt][rg] >> (8 * i)) & 0xffu];
                                o[i] = (_Float16)v;
                            }
                            const u32x2 ow = __builtin_bit_cast(u32x2, o);
                            w[e][0] = ow[0];
                            w[e][1] = ow[1];
                        }
                        const auto s0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                        const auto s1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                        const u32x4 v = {s0[0], s1[0], s0[1], s1[1]};
                        if (tl < nv) *reinterpret_cast<u32x4 *>(yrow + 32 * pt + 16 * j) = v;
                    }
            };
            for (int c = c_begin; c < c_end; ++c) {
                const int buf = (c - c_begin) & 1;
                const unsigned char *set = smem + buf * LY::kSet;
                const float *s_loc = reinterpret_cast<const float *>(set + LY::kOffLoc);
                const float *s_tot = reinterpret_cast<const float *>(set + LY::kOffTot);
                new_lane();
                const int tl = tb * kBlk + l32;
                i32x4 ct[4];
                if (LY::kOneC) {
                    load_c_rows(buf, tb, ct);
                    done(8 + tb, c - c_begin + 1);
                }
                if (c > c_begin) epilogue(c - 1, buf ^ 1);
                if (tb * kBlk < min(kQ, L - c * kQ)) {
                    if (!LY::kOneC) load_c_rows(buf, tb, ct);
                    const float loc_t = s_loc[tl];
                    i32x16 gi;
                    if (PT == 1) gi = score_tile(set, mid, ct);
                    // the skip term: D x as a product with a diagonal matrix
                    if (PT == 2) {
                        diagonal(d16, skip);
                        diagonal(d16_rest, skip_rest);
                    }
                    f16x8 x0[PT], x1[PT];
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt) {
                        x0[pt] = load_x(set, tb * kBlk, pt);
                        x1[pt] = load_x(set, tb * kBlk + 16, pt);
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0[pt], skip_rest[0], (f32x16)(0.0f), 0, 0, 0);
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[pt], skip_rest[1], acc[pt], 0, 0, 0);
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0[pt], skip[0], acc[pt], 0, 0, 0);
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[pt], skip[1], acc[pt], 0, 0, 0);
                    }
                    if (PT == 2) {
                        new_lane();
                        gi = score_tile(set, mid, ct);
                    }
                    off_diagonal(set, tb, mid, tb, true, loc_t, ct, gi, acc);
                    if (PT == 2) new_lane();
                    // diagonal block pair: per-element decay, causal mask on the narrowed values
                    const bool factored = __builtin_amdgcn_readfirstlane(-s_tot[tb] < 64.0f);
                    f16x4 lq[4];
                    if (factored) {
                        const float *s_w2 = reinterpret_cast<const float *>(set + LY::kOffW2);
                        const float e_row = exp2_fast(loc_t);
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg) {
                            const f32x4 w4 = *reinterpret_cast<const f32x4 *>(s_w2 + tb * kBlk + 8 * rg + 4 * hb);
#pragma unroll
                            for (int i = 0; i < 4; ++i) lq[rg][i] = (_Float16)((float)gi[4 * rg + i] * (e_row * w4[i]));
                        }
                    } else {
                        const float *s_dt = reinterpret_cast<const float *>(set + LY::kOffDt);
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg) {
                            const f32x4 cs4 = *reinterpret_cast<const f32x4 *>(s_loc + tb * kBlk + 8 * rg + 4 * hb);
                            const f32x4 ds4 = *reinterpret_cast<const f32x4 *>(s_dt + tb * kBlk + 8 * rg + 4 * hb);
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                lq[rg][i] = (_Float16)((float)gi[4 * rg + i] * (exp2_fast(loc_t - cs4[i]) * ds4[i]));
                        }
                    }
                    if (PT == 2) {
                        keep[0] = s_keep[32 * hb + l32];
                        keep[1] = s_keep[64 + 32 * hb + l32];
                    }
                    u32x4 l0 = __builtin_bit_cast(u32x4, __builtin_shufflevector(lq[0], lq[1], 0, 1, 2, 3, 4, 5, 6, 7));
                    u32x4 l1 = __builtin_bit_cast(u32x4, __builtin_shufflevector(lq[2], lq[3], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        l0[k] &= keep[0][k];
                        l1[k] &= keep[1][k];
                    }
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt) {
                        if (PT == 2) {  // (with 32 channels the operands are still in registers)
                            x0[pt] = load_x(set, tb * kBlk, pt);
                            x1[pt] = load_x(set, tb * kBlk + 16, pt);
                        }
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0[pt], __builtin_bit_cast(f16x8, l0), acc[pt], 0, 0, 0);
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[pt], __builtin_bit_cast(f16x8, l1), acc[pt], 0, 0, 0);
                    }
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg) {
                            if (GATED)
                                zq[pt][rg] = *reinterpret_cast<const uint32_t *>(set + LY::kOffZs + tl * kZsStride + 32 * pt +
                                                                                 8 * rg + 4 * hb);
                            if (!d_by_mfma) {
                                const int row = tok_pos(tl);
                                xq[pt][rg] = *reinterpret_cast<const f16x4 *>(set + LY::kOffXs + row * kXsStride * 2 +
                                                                              x_part<PT>(row, 2 * pt + (rg >> 1), 2 * (rg & 1) + hb));
                            }
                        }
                }
                __syncthreads();  // the next chunk is staged; this one's early terms are in LDS
            }
            if (tb * kBlk < L - (c_end - 1) * kQ) epilogue(c_end - 1, (c_end - 1 - c_begin) & 1);
        } else {
            // ---- the early terms of block 3 - wave: the carried state and the first block pairs; the wave of block 0, which
            // has no pairs, also turns the next chunk's step sizes into its token weights ----
            const int tb = kNBlk - 1 - wave, mid = tb >= 2 ? tb - 1 : tb;
            float dt0, dt1;
            if (tb == 0) load_dt(c_begin, dt0, dt1);
            const bool over = starts_over();
            if (tb == 0) {
                if (over) load_dt(c_begin, dt0, dt1);
                token_weights(c_begin, smem, dt0, dt1);
                if (c_begin + 1 < c_end) load_dt(c_begin + 1, dt0, dt1);
            }
            if (convert_init) __syncthreads();
            __syncthreads();  // the first chunk is staged
            for (int c = c_begin; c < c_end; ++c) {
                const int buf = (c - c_begin) & 1;
                const unsigned char *set = smem + buf * LY::kSet;
                const float *s_cum = reinterpret_cast<const float *>(set + LY::kOffCum);
                const float *s_loc = reinterpret_cast<const float *>(set + LY::kOffLoc);
                new_lane();
                if (tb == 0 && c + 1 < c_end) {
                    token_weights(c + 1, smem + (buf ^ 1) * LY::kSet, dt0, dt1);
                    if (c + 2 < c_end) load_dt(c + 2, dt0, dt1);
                }
                if (tb * kBlk < min(kQ, L - c * kQ)) {
                    const int tl = tb * kBlk + l32;
                    i32x4 ct[4];
                    load_c_rows(buf, tb, ct);
                    if (LY::kOneC) done(12 + tb, c - c_begin + 1);
                    const float loc_t = s_loc[tl], cum_t = s_cum[tl];
                    const float r_tb = tb > 0 ? s_cum[tb * kBlk - 1] : 0.0f;
                    const int sb0 = first_alive(s_cum, tb, r_tb);
                    i32x16 gi;
                    if (sb0 < mid) gi = score_tile(set, sb0, ct);
                    f32x16 acc[PT];
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt) acc[pt] = (f32x16)(0.0f);
                    if (!__builtin_amdgcn_readfirstlane(r_tb < -dead)) {
                        // carried state: Y^T[p,t] = exp(cum_t) sum_n H[p,n] Cq[t,n]
                        const _Float16 *s_hs = reinterpret_cast<const _Float16 *>(h_rows(buf)) + l32 * kHsStride + 16 * hb;
#pragma unroll
                        for (int k8 = 0; k8 < 8; ++k8) {
                            f16x8 hf[PT];
#pragma unroll
                            for (int pt = 0; pt < PT; ++pt)
                                hf[pt] = *reinterpret_cast<const f16x8 *>(s_hs + 32 * pt * kHsStride + 32 * (k8 >> 1) + 8 * (k8 & 1));
                            const i32x4 c4 = ct[k8 >> 1];
                            const f16x8 cf = i8x8_to_f16((uint32_t)c4[2 * (k8 & 1)], (uint32_t)c4[2 * (k8 & 1) + 1]);
#pragma unroll
                            for (int pt = 0; pt < PT; ++pt)
                                acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[pt], cf, acc[pt], 0, 0, 0);
                        }
                        const float e_t = exp2_fast(cum_t) * kAcc;
#pragma unroll
                        for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                            for (int r = 0; r < 16; ++r) acc[pt][r] *= e_t;
                    }
                    if (LY::kOneH) done(4 + tb, c - c_begin + 1);
                    off_diagonal(set, tb, sb0, mid, false, loc_t, ct, gi, acc);
                    f32x4 *part = part_of(buf) + tb * PT * 4 * 64 + 32 * hb + l32;
                    if (LY::kOnePart) wait_done(tb, c - c_begin);
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg)
                            part[(pt * 4 + rg) * 64] =
                                (f32x4){acc[pt][4 * rg], acc[pt][4 * rg + 1], acc[pt][4 * rg + 2], acc[pt][4 * rg + 3]};
                } else if (PT == 2) {  // a block past the end (of the last chunk) reads nothing
                    done(4 + tb, c - c_begin + 1);
                    if (LY::kOneC) done(12 + tb, c - c_begin + 1);
                }
                __syncthreads();
            }
        }
    } else if (role == 2) {
        // ================= state waves =================
        // st[pt][r]: p = 32 pt + l32, n = 32 wave + 8 (r/4) + 4 hb + r%4, as in prefill_mfma_kernel
        f32x16 st[PT];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) st[pt] = (f32x16)(0.0f);
        // the lane's row of the caller's states, where it is read and where it is written: kept over the chunks it would not fit
        auto st_row = [&]() {
            new_lane();
            return ((size_t)bh * kP + p_base + l32) * kN + 32 * wave + 4 * hb;
        };
        if constexpr (SHARED) {
            if (c_begin > 0) {
                if (wave == 0 && lane == 0) *s_left = await_left(a, cut, left_count(a, cut));
                if (!starts_over()) read_left_state(a, cut, wave, lane, st);
            }
        }
        if (SEG && seg > 0) {
            // the combination of the earlier segments' states, see prefill_mfma_kernel
            const size_t pairs = (size_t)a.s.batch * H;
            auto add_segment = [&](int j, float w) {
#pragma unroll
                for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(
                            a.seg_state + segment_state_at((size_t)j * pairs + bh, half + pt, wave, rg, lane));
#pragma unroll
                        for (int i = 0; i < 4; ++i) st[pt][4 * rg + i] = fmaf(w, v[i], st[pt][4 * rg + i]);
                    }
            };
            const SegmentsInFront front(a, seg, pairs, bh);
            add_segment(seg - 1, 1.0f);
            float dsum = front.decay(seg - 1);
            for (int j = seg - 2; j >= 0; --j) {
                if (dsum < -dead && front.cannot_count(dsum, Ah, st)) {
                    if (!a.init_state) break;
                    for (; j > 0; --j) dsum += front.decay(j);
                }
                add_segment(j, exp2_fast(dsum));
                dsum += front.decay(j);
            }
        }
        if (convert_init) {
            __syncthreads();  // the scales are in LDS
            const float *init = a.init_state + st_row();
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const float inv = kNarrow * (d_by_mfma ? y_scale : 1.0f) / (s_sx[32 * pt + l32] * sB);
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(init + 32 * pt * kN + 8 * rg);
#pragma unroll
                    for (int i = 0; i < 4; ++i) st[pt][4 * rg + i] = v[i] * inv;
                }
            }
        }
        auto publish = [&](int buf) {  // the state as fp16, operand of the next chunk's C.H product
            unsigned char *row = h_rows(buf) + (l32 * kHsStride + 32 * wave + 4 * hb) * 2;
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    f16x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = (_Float16)st[pt][4 * rg + i];
                    *reinterpret_cast<f16x4 *>(row + 32 * pt * kHsStride * 2 + 16 * rg) = v;
                }
        };
        publish(0);
        __syncthreads();  // the first chunk is staged
        const bool want_state = a.state && c_end == nchunks, leave = SHARED && c_end < nchunks;
        for (int c = c_begin; c < c_end; ++c) {
            const int buf = (c - c_begin) & 1;
            const unsigned char *set = smem + buf * LY::kSet;
            const float *s_cum = reinterpret_cast<const float *>(set + LY::kOffCum);
            const float *s_tot = reinterpret_cast<const float *>(set + LY::kOffTot);
            if (c + 1 < c_end || want_state || leave) {
                new_lane();
                const int i16 = l32 & 15, c16 = l32 >> 4;
                const unsigned char *bq_src =
                    set + LY::kOffBq + (8 * hb + (i16 >> 1)) * kBqStride + 32 * wave + 16 * c16 + 8 * (i16 & 1);
                const int xr = 8 * hb + (i16 >> 2);
                const unsigned char *xs_src = set + LY::kOffXs + xr * kXsStride * 2;
                const _Float16 *s_ws = reinterpret_cast<const _Float16 *>(set + LY::kOffWs) + 8 * hb;
                const _Float16 *s_wd = reinterpret_cast<const _Float16 *>(set + LY::kOffWd) + 8 * hb;
                struct Ops {
                    u32x2 bw;
                    f16x8 x[PT], wv, wd;
                };
                auto fetch = [&](int step, Ops &o) {
                    const int row = 16 * step;
                    o.bw = lds_read_tr8(bq_src + row * kBqStride);
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
                        o.x[pt] = lds_read_tr16x8<kXsStride>(xs_src + row * kXsStride * 2 +
                                                             x_part<PT>(xr, 2 * pt + c16, i16 & 3));
                    o.wv = *reinterpret_cast<const f16x8 *>(s_ws + row);
                    if (PRECISE) o.wd = *reinterpret_cast<const f16x8 *>(s_wd + row);
                };
                auto decay = [&](float log2_dec) {
                    const float dec = exp2_fast(log2_dec);
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) st[pt][r] *= dec;
                };
                auto add = [&](const Ops &o) {
                    const f16x8 bf = i8x8_to_f16(o.bw[0], o.bw[1]) * o.wv;
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
                        st[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, o.x[pt], st[pt], 0, 0, 0);
                    if (PRECISE) {
                        const f16x8 rest = bf * o.wd;
#pragma unroll
                        for (int pt = 0; pt < PT; ++pt)
                            st[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rest, o.x[pt], st[pt], 0, 0, 0);
                    }
                };
                // What a block adds decays by exp2(cum_last - m) before the chunk ends; the dead blocks are the first ones and
                // only decay.  A chunk without dead blocks runs as straight code, so that its LDS reads, conversions and
                // products overlap.
                const float cum_last = s_cum[kQ - 1], m0 = s_cum[kBlk - 1], m1 = s_cum[2 * kBlk - 1], m2 = s_cum[3 * kBlk - 1];
                const f32x4 tot = *reinterpret_cast<const f32x4 *>(s_tot);
                const int first = __builtin_amdgcn_readfirstlane((cum_last - m0 < -dead) + (cum_last - m1 < -dead) +
                                                                 (cum_last - m2 < -dead));
                if (!PRECISE) decay(cum_last);
                if (first == 0) {
                    Ops ops[2];
                    fetch(0, ops[0]);
#pragma unroll
                    for (int step = 0; step < 2 * kNBlk; ++step) {
                        if (step + 1 < 2 * kNBlk) fetch(step + 1, ops[(step + 1) & 1]);
                        if (PRECISE && (step & 1) == 0) decay(tot[step >> 1]);  // the block's own total (0 past the end)
                        add(ops[step & 1]);
                    }
                } else {
                    if (PRECISE) decay(first == 1 ? tot[0] : first == 2 ? tot[0] + tot[1] : tot[0] + tot[1] + tot[2]);
                    for (int sb = first; sb < kNBlk; ++sb) {
                        Ops o0, o1;
                        fetch(2 * sb, o0);
                        fetch(2 * sb + 1, o1);
                        if (PRECISE) decay(s_tot[sb]);
                        add(o0);
                        add(o1);
                    }
                }
                if (c + 1 < c_end) {
                    if (LY::kOneH) {
#pragma unroll
                        for (int k = 0; k < kNBlk; ++k) wait_done(4 + k, c - c_begin + 1);
                    }
                    publish(buf ^ 1);
                }
            }
            __syncthreads();
        }
        if constexpr (SHARED)
            if (leave) leave_state(a, cut, wave, lane, st);  // for the piece behind
        if (want_state) {
            float *state = a.state + st_row();
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const float sc = s_sx[32 * pt + l32] * sB / ((d_by_mfma ? y_scale : 1.0f) * kNarrow);
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    f32x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = st[pt][4 * rg + i] * sc;
                    *reinterpret_cast<f32x4 *>(state + 32 * pt * kN + 8 * rg) = v;
                }
            }
        }
    } else {
        // ================= staging waves =================
        // A thread takes tokens r0 + 32 k of a chunk, of each 4 channels of x and z and 16 states of B and C (8 lanes cover a
        // row, a wave 8 consecutive rows).
        const int r0 = tid4 >> 3, p8 = tid4 & 7;
        const uint32_t x_off = r0 * x_row + (uint32_t)(4 * PT) * p8, b_off = r0 * b_row + 16u * p8;
        xvec xr[4], zr[4];
        u32x4 br[4], cr[4];
        auto issue_loads = [&](int c) {
            const size_t tok = (size_t)b * L + c * kQ;
            const int8_t *xbase = a.x + (tok * H + h) * kP + p_base, *bbase = a.B + (tok * G + g) * kN;
            const int8_t *zbase = a.z + (tok * H + h) * kP + p_base, *cbase = a.C + (tok * G + g) * kN;
            const int nv = min(kQ, L - c * kQ);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                size_t xk = (size_t)(kBlk * k) * x_row, bk = (size_t)(kBlk * k) * b_row;  // uniform
                uint32_t xo = x_off, bo = b_off;
                if (nv < kQ) {  // rows past the end are read from the last row and zeroed where they are stored
                    const uint32_t row = (uint32_t)min(r0 + kBlk * k, nv - 1);
                    xk = bk = 0;
                    xo = row * x_row + (uint32_t)(4 * PT) * p8;
                    bo = row * b_row + 16u * p8;
                }
                xr[k] = *reinterpret_cast<const xvec *>(xbase + xk + xo);
                if (GATED) zr[k] = *reinterpret_cast<const xvec *>(zbase + xk + xo);
                br[k] = *reinterpret_cast<const u32x4 *>(bbase + bk + bo);
                cr[k] = *reinterpret_cast<const u32x4 *>(cbase + bk + bo);
            }
        };
        auto stage = [&](int c, int buf) {
            unsigned char *set = smem + buf * LY::kSet;
            const int nv = min(kQ, L - c * kQ), row0 = tok_pos(r0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (nv < kQ && r0 + kBlk * k >= nv) {
                    xr[k] = (xvec)(0u);
                    br[k] = cr[k] = (u32x4){0u, 0u, 0u, 0u};
                }
                const int row = row0 + kBlk * k, tok = r0 + kBlk * k;
                unsigned char *xs_row = set + LY::kOffXs + row * kXsStride * 2;
#pragma unroll
                for (int q = 0; q < PT; ++q)
                    *reinterpret_cast<f16x4 *>(xs_row + x_part<PT>(row, p8 * PT >> 2, (p8 * PT & 3) + q)) = i8x4_to_f16_xs(xr[k][q]);
                if (GATED) *reinterpret_cast<xvec *>(set + LY::kOffZs + tok * kZsStride + 4 * PT * p8) = zr[k];
                *reinterpret_cast<u32x4 *>(set + LY::kOffBq + row * kBqStride + 16 * p8) = br[k];
                if (!LY::kOneC) *reinterpret_cast<u32x4 *>(c_rows(buf) + tok * kN + 16 * (p8 ^ (r0 & 7))) = cr[k];
            }
            if (LY::kOneC) {
                if (c > c_begin) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) wait_done(8 + k, c - c_begin);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<u32x4 *>(c_rows(0) + (r0 + kBlk * k) * kN + 16 * (p8 ^ (r0 & 7))) = cr[k];
            }
        };
        issue_loads(c_begin);
        if (starts_over()) issue_loads(c_begin);
        if (convert_init) __syncthreads();
        stage(c_begin, 0);
        if (c_begin + 1 < c_end) issue_loads(c_begin + 1);
        __syncthreads();  // the first chunk is staged
        for (int c = c_begin; c < c_end; ++c) {
            if (c + 1 < c_end) {
                stage(c + 1, (c + 1 - c_begin) & 1);
                if (c + 2 < c_end) issue_loads(c + 2);
            }
            __syncthreads();
        }
    }
}

template <bool PRECISE, int PT, bool GATED, Walk WALK>
hipError_t launch_walk(const typename WalkArgs<WALK>::type &a, unsigned workgroups, hipStream_t stream)
{
    const hipError_t e = allow_full_lds<prefill_wide_kernel<PRECISE, PT, GATED, WALK>>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((prefill_wide_kernel<PRECISE, PT, GATED, WALK>), dim3(workgroups), dim3(kWideThreads), (WideLds<PT, GATED>::kBytes),
                       stream, a);
    return hipGetLastError();
}

template <bool PRECISE, int PT, bool GATED>
hipError_t launch(const SsdArgs &a, hipStream_t stream)
{
    const unsigned wgs = (unsigned)((2 / PT) * a.s.batch * a.s.nheads);
    if (a.nseg > 1) return launch_walk<PRECISE, PT, GATED, Walk::segment>(a, wgs * a.nseg, stream);
    return launch_walk<PRECISE, PT, GATED, Walk::whole>(a, wgs, stream);
}

}  // namespace

hipError_t launch_prefill_wide(const SsdArgs &a, bool halves, bool precise, hipStream_t stream)
{
    if (!halves) {
        if (precise) return a.z ? launch<true, 2, true>(a, stream) : launch<true, 2, false>(a, stream);
        return a.z ? launch<false, 2, true>(a, stream) : launch<false, 2, false>(a, stream);
    }
    if (precise) return a.z ? launch<true, 1, true>(a, stream) : launch<true, 1, false>(a, stream);
    return a.z ? launch<false, 1, true>(a, stream) : launch<false, 1, false>(a, stream);
}

hipError_t launch_prefill_wide_shared(const SharedArgs &a, bool precise, hipStream_t stream)
{
    const unsigned wgs = (unsigned)(a.rounds.steps * a.rounds.groups);
    if (precise)
        return a.z ? launch_walk<true, 2, true, Walk::shared>(a, wgs, stream) : launch_walk<true, 2, false, Walk::shared>(a, wgs, stream);
    return a.z ? launch_walk<false, 2, true, Walk::shared>(a, wgs, stream) : launch_walk<false, 2, false, Walk::shared>(a, wgs, stream);
}

}  // namespace quamba
