// Tiles, operand layouts and scales shared by the matrix-core prefill kernels (prefill_mfma.hip describes the arithmetic).
#pragma once
#include "quamba_internal.h"

namespace quamba {

// What a workgroup walks of its sequence: all of it, a segment of a sequence split (see SsdArgs), or a piece of shared rounds.
enum class Walk { whole, segment, shared };

// Shared rounds: launches of a few more (sequence, head) pairs than the device holds workgroups.  See shared_rounds (prefill_mfma.hip).
struct SharedRounds {
    static constexpr int kPlaces = 8;  // of a group: workgroups that share its pairs
    struct Piece {
        int c_begin, c_end;  // chunks
        int16_t pair;        // of the group, behind the lead
        int16_t cut;         // at the piece's end or start
    };
    bool wide;    // places are compute units, each with a workgroup of 16 waves; otherwise half units, of 8 waves
    int groups;   // workgroup i: step i / groups of the list of group i % groups
    int lead;     // steps that are whole pairs, in front of the pieces
    int steps;    // in all; 0: the launch is not of this kind
    int polls;    // of a wait for the piece in front
    float *state; // [cut][group][headdim * d_state]: the accumulators at the cuts
    int *left;    // [cut][group]: waves that have left their part of them there
    Piece piece[2 * kPlaces + kPlaces - 2];
};
struct SharedArgs : SsdArgs {
    SharedRounds rounds;
};
template <Walk WALK>
struct WalkArgs {
    typedef SsdArgs type;
};
template <>
struct WalkArgs<Walk::shared> {
    typedef SharedArgs type;
};

hipError_t launch_prefill_wide_shared(const SharedArgs &a, bool precise, hipStream_t stream);

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kP = 64, kN = 128, kQ = 128, kBlk = 32, kNBlk = kQ / kBlk;
constexpr int kHsStride = 136;  // halves per row of H [p][n]
constexpr int kBqStride = 144;  // bytes per row of Bq [token][n]
constexpr float kNarrow = 1.0f / 128.0f;  // applied to G and H before narrowing to fp16; undone in the epilogue
// Scales that keep every fp16 operand in the normal range.  x is staged as fp16 codes times kXs; the output
// accumulators hold the output in code units times 2^-7 kAcc; the state accumulators the state times 2^-7 (kNarrow).
// Hence the token weights on the score columns carry kAcc / kXs = 1/4 (score tiles, up to 2^14 after their own 2^-7,
// times dt / 4 stay finite for dt up to 16), those on the rows of B carry kNarrow / kXs = 1/8 (dt / 8 times the decay
// is far from the subnormals), and the C operand of the carried-state product carries kAcc.
constexpr float kXs = 1.0f / 16.0f;
constexpr float kAcc = 1.0f / 64.0f;
// A product whose operands are separated by a decay factor below 2^-kDead (prefix sums are in log2 units) is left out
// unless the caller asks for it: it is below 2.4e-10 of the term's own undecayed size.
constexpr float kDead = 32.0f;

// 2^x by the hardware instruction (prefix sums are carried in log2 units, so no multiply by log2 e is needed).
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Lane index recomputed where it is called: the mask passes through an empty asm statement, so the compiler can neither
// hoist the result out of a loop nor keep it in a register across one.
__device__ __forceinline__ int fresh_lane() {
    unsigned m = ~0u;
    asm volatile("" : "+s"(m));
    return (int)__builtin_amdgcn_mbcnt_hi(m, __builtin_amdgcn_mbcnt_lo(m, 0u));
}
// LDS row of token s of the chunk: bits 2 and 3 swapped (prefill_mfma.hip says why).
__device__ __forceinline__ int tok_pos(int s) { return (s & ~12) | ((s & 4) << 1) | ((s & 8) >> 1); }

// Transposing LDS loads.  Inside each group of 16 lanes, result byte j of lane i comes from the 8 bytes addressed by
// lane 2j + (i >> 3), byte i & 7 (8-bit form); result half j of lane i from the 8 bytes addressed by lane
// 4j + (i >> 2), half i & 3 (16-bit form).  With source lane 2j + q pointing at (token row j, 8 columns starting at
// 8q), resp. 4j + q at (token row j, 4 columns starting at 4q), lane i receives column i of 8 (resp. 4) token rows:
// the layout of an MFMA operand whose k index is the token.
typedef int v2i_lds __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 lds_read_tr8(const unsigned char *p)
{
    return __builtin_bit_cast(
        u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i_lds *)(p)));
}
__device__ __forceinline__ f16x4 lds_read_tr16(const unsigned char *p)
{
    typedef short v4s_lds __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(
        f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_lds *)(p)));
}
// 8 tokens x one column of fp16 x (two 4-token transposing loads, token rows r .. r+7 of the lane group)
template <int PITCH_HALVES>
__device__ __forceinline__ f16x8 lds_read_tr16x8(const unsigned char *p)
{
    const f16x4 lo = lds_read_tr16(p), hi = lds_read_tr16(p + 4 * 2 * PITCH_HALVES);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// 8 int8 codes (two dwords, lowest address first) -> 8 exact fp16 values, one conversion per code: the source byte is
// picked and sign-extended by the instruction's sub-dword source select, the result written to the low or high half of
// the destination by its destination select (the high half keeps the low one).
__device__ __forceinline__ uint32_t i8x2_to_f16_lo_hi(uint32_t w, int first_byte)
{
    uint32_t r;
    if (first_byte == 0) {
        asm("v_cvt_f16_i16_sdwa %0, sext(%1) dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:BYTE_0" : "=v"(r) : "v"(w));
        asm("v_cvt_f16_i16_sdwa %0, sext(%1) dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1" : "+v"(r) : "v"(w));
    } else {
        asm("v_cvt_f16_i16_sdwa %0, sext(%1) dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:BYTE_2" : "=v"(r) : "v"(w));
        asm("v_cvt_f16_i16_sdwa %0, sext(%1) dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3" : "+v"(r) : "v"(w));
    }
    return r;
}
__device__ __forceinline__ f16x8 i8x8_to_f16(uint32_t w0, uint32_t w1)
{
    const u32x4 r = {i8x2_to_f16_lo_hi(w0, 0), i8x2_to_f16_lo_hi(w0, 2), i8x2_to_f16_lo_hi(w1, 0),
                     i8x2_to_f16_lo_hi(w1, 2)};
    return __builtin_bit_cast(f16x8, r);
}

// 4 int8 codes (one dword) -> fp16 values kXs * code, exact: byte^0x80 placed under the fp16 pattern of 64 (whose
// last mantissa bit weighs 1/16) gives 64 + (code + 128) / 16; subtract 72.
__device__ __forceinline__ f16x4 i8x4_to_f16_xs(uint32_t w)
{
    static_assert(kXs == 1.0f / 16.0f, "the bit pattern below encodes a step of 1/16");
    const f16x2 bias = {(_Float16)72.0f, (_Float16)72.0f};
    w ^= 0x80808080u;
    union { f16x4 v; f16x2 h[2]; } r;
    r.h[0] = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x54545454u, w, 0x04010400u)) - bias;
    r.h[1] = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x54545454u, w, 0x04030402u)) - bias;
    return r.v;
}

template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, BOUND));
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves only (no LDS round trips):
// shifts by 1, 2, 4, 8 inside each row of 16 lanes (zero fill), then the last lane of row 0/2 is added to row 1/3
// and the last lane of row 1 to rows 2 and 3.
// `row` receives the scan inside the lane's row of 16 lanes alone (the first four steps).
__device__ __forceinline__ float wave_inclusive_scan(float v, float &row)
{
    v += dpp_f32<0x111, 0xf, true>(v);   // row_shr:1
    v += dpp_f32<0x112, 0xf, true>(v);   // row_shr:2
    v += dpp_f32<0x114, 0xf, true>(v);   // row_shr:4
    v += dpp_f32<0x118, 0xf, true>(v);   // row_shr:8
    row = v;
    v += dpp_f32<0x142, 0xa, false>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_f32<0x143, 0xc, false>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Sum of the values of the lanes behind this one inside its row of 16 lanes (0 for the row's last lane): row shifts
// towards lower lanes with zero fill.  Unlike the difference of two prefix sums it carries no rounding error of the
// size of the sums in front of the lane.
__device__ __forceinline__ float row_suffix_sum_exclusive(float v)
{
    float s = dpp_f32<0x101, 0xf, true>(v);  // row_shl:1
    s += dpp_f32<0x101, 0xf, true>(s);
    s += dpp_f32<0x102, 0xf, true>(s);       // row_shl:2
    s += dpp_f32<0x104, 0xf, true>(s);       // row_shl:4
    s += dpp_f32<0x108, 0xf, true>(s);       // row_shl:8
    return s;
}

__device__ __forceinline__ f16x8 pack_f16x8(const float v[8])
{
    f16x8 r;
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = (_Float16)v[j];
    return r;
}

// A segment's end state in the workspace, where the state pass writes and the outputs' kernels read it: as it stands in the
// accumulators, 4 values of a lane behind those of the lane before, so that a wave moves 1 KB of consecutive memory at once.  (In
// the order [p][n] of the caller's states it touches 32 lines of 32 bytes each: 1.2 us per segment and workgroup.)  Wave w's values
// 4 rg .. 4 rg + 3 of the channels 32 q .. 32 q + 31 lie behind the returned offset.
__device__ __forceinline__ size_t segment_state_at(size_t pair, int q, int wave, int rg, int lane)
{
    return pair * (kP * kN) + (size_t)(((q * 4 + wave) * 4 + rg) * 64 + lane) * 4;
}

constexpr int kMaxSegments = 9;  // of the sequence split

// The segments in front of one: their decays, one to a lane, and where the walk back over their states may end.  The states come
// from memory one after the other, and the segment's first chunk waits for them: of 24 heads, 2048 tokens in 8 segments, with decays of
// 2^-14 a chunk and more, two or three of up to seven are read, which takes 1.5 us less than all.
// The walk ends where the rest cannot change a bit of the sum: half a unit in a value's last place is more than 2^-25 of it, and a state
// that its segment began at zero is, in accumulator units, at most the largest codes' product times the sum of the segment's step
// sizes, which its decay gives (dt >= 0; up to 1024, far from where an operand in fp16 could overflow).  An end at a share of the
// undecayed size (2^-32: 19.5 us instead of 19.7, 5 segments of a chunk 10.2 instead of 10.5) would lose what stands beside zeros or far smaller
// values.  The segment of the caller's initial state, of any size or not finite, is always read.
struct SegmentsInFront {
    float mine;
    __device__ __forceinline__ SegmentsInFront(const SsdArgs &a, int seg, size_t pairs, int bh)
        : mine(a.seg_decay[(size_t)min((int)threadIdx.x & 63, seg - 1) * pairs + bh])
    {
    }
    __device__ __forceinline__ float decay(int j) const
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), j));
    }
    template <int PT>
    __device__ __forceinline__ bool cannot_count(float log2_decay, float Ah, const f32x16 (&st)[PT]) const
    {
        static_assert(kMaxSegments <= 16, "a row of lanes");
        float lowest = mine;
        lowest = fminf(lowest, dpp_f32<0x128, 0xf, true>(lowest));  // row_ror
        lowest = fminf(lowest, dpp_f32<0x124, 0xf, true>(lowest));
        lowest = fminf(lowest, dpp_f32<0x122, 0xf, true>(lowest));
        lowest = fminf(lowest, dpp_f32<0x121, 0xf, true>(lowest));
        float least = __builtin_inff();
#pragma unroll
        for (int pt = 0; pt < PT; ++pt)
#pragma unroll
            for (int r = 0; r < 16; ++r) least = fminf(least, fabsf(st[pt][r]));
        constexpr float margin = 2.0f;  // over what rounding adds to the sums
        const float largest = exp2_fast(log2_decay) * lowest * (margin * kNarrow * 0x1p14f * 0x1p25f);  // times Ah, as below
        return __all(mine <= 0.0f && Ah < 0.0f && lowest >= 1024.0f * Ah && largest > least * Ah);
    }
};

// Where a piece of shared rounds leaves its accumulators in the workspace.  They are stored and loaded at device scope, past the
// caches of the XCD, on whichever of them the piece behind runs: a release fence would write back the XCD's whole cache, and
// 448 of them took 80 us of a launch.
constexpr int kDeviceScope = 16;  // the instructions' SC1 bit
__device__ __forceinline__ auto left_state(const SharedArgs &a, int cut)
{
    return __builtin_amdgcn_make_buffer_rsrc(a.rounds.state + (size_t)cut * (kP * kN), 0, 4 * kP * kN, 0x00020000);
}
__device__ __forceinline__ int left_at(int pt, int wave, int rg, int lane) { return (int)(4 * segment_state_at(0, pt, wave, rg, lane)); }
template <int PT>
__device__ __forceinline__ void read_left_state(const SharedArgs &a, int cut, int wave, int lane, f32x16 (&st)[PT])
{
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const f32x4 v = __builtin_bit_cast(
                f32x4, __builtin_amdgcn_raw_buffer_load_b128(left_state(a, cut), left_at(pt, wave, rg, lane), 0, kDeviceScope));
#pragma unroll
            for (int i = 0; i < 4; ++i) st[pt][4 * rg + i] = v[i];
        }
}
// ... and a count for each of the four waves that hold them.
template <int PT>
__device__ __forceinline__ void leave_state(const SharedArgs &a, int cut, int wave, int lane, const f32x16 (&st)[PT])
{
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = st[pt][4 * rg + i];
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), left_state(a, cut), left_at(pt, wave, rg, lane), 0,
                                                   kDeviceScope);
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores have been performed
    if (lane == 0) __hip_atomic_fetch_add(a.rounds.left + cut, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int left_count(const SharedArgs &a, int cut)
{
    return __hip_atomic_load(a.rounds.left + cut, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The piece goes on from the accumulators that the piece in front of it leaves.  That one waits for nobody, and its workgroup
// comes well in front of this one.  Should it not be there after some milliseconds all the same (false), the walk begins at the
// sequence's start, which gives the same results.  n: the count as it was last seen.
__device__ __forceinline__ bool await_left(const SharedArgs &a, int cut, int n)
{
    for (int i = 0; n < 4 && i < a.rounds.polls; ++i) {
        __builtin_amdgcn_s_sleep(8);
        n = left_count(a, cut);
    }
    return n >= 4 && a.rounds.polls >= 0;  // (below zero, in tests: as if it never came)
}
// The piece of a workgroup, false if it has none (a group may have one pair less).
__device__ __forceinline__ bool shared_piece(const SharedArgs &a, int &pair, int &cut, int &c_begin, int &c_end)
{
    const int step = (int)blockIdx.x / a.rounds.groups, group = (int)blockIdx.x - step * a.rounds.groups;
    pair = step;
    if (step >= a.rounds.lead) {
        const SharedRounds::Piece piece = a.rounds.piece[step - a.rounds.lead];
        pair = a.rounds.lead + piece.pair;
        c_begin = piece.c_begin;
        c_end = piece.c_end;
        cut = piece.cut * a.rounds.groups + group;
    }
    pair = pair * a.rounds.groups + group;
    return pair < a.s.batch * a.s.nheads;
}

// Workgroup -> (sequence, head).  Hardware hands consecutive workgroup ids to the 8 XCDs round-robin, each XCD with
// its own L2.  When the number of (sequence, state group) units is a multiple of 8, all heads of a unit are put on
// one XCD, so that the B and C rows they share are fetched into one L2 instead of eight.
__device__ __forceinline__ int block_to_bh(const SsdArgs &a, int i)
{
    const int H = a.s.nheads, G = a.s.ngroups, hpg = H / G;
    const int units = a.s.batch * G;
    if (units % 8 != 0) return i;
    const int x = i & 7, slot = i >> 3;
    const int u = x + 8 * (slot / hpg), hl = slot % hpg;
    const int b = u / G, g = u - b * G;
    return b * H + g * hpg + hl;
}

// The same map in the kernels of short batches, by reciprocals.
__device__ __forceinline__ void place_of(const SsdArgs &a, int i, int &b, int &h, int &g)
{
    const int H = a.s.nheads, G = a.s.ngroups, hpg = a.heads_per_group;
    const bool by_units = a.s.batch * G % 8 == 0;
    const int slot = i >> 3, turn = quotient(slot, a.inv_heads_per_group), u = (i & 7) + 8 * turn;
    b = quotient(by_units ? u : i, by_units ? a.inv_groups : a.inv_heads);
    const int rest = (by_units ? u : i) - b * (by_units ? G : H);  // the group, or the head
    g = by_units ? rest : quotient(rest, a.inv_heads_per_group);
    h = by_units ? rest * hpg + slot - turn * hpg : rest;
}

}  // namespace
}  // namespace quamba
