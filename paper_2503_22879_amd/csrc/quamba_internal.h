// Internal launch interface between the C-ABI layer and the HIP kernels (not installed).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>

#include "quamba_ssd.h"

namespace quamba {

// ---- host helpers of the launchers ----
constexpr size_t kLdsPerCu = 160 * 1024;  // LDS of one gfx950 compute unit

// Compute units of the current device (asked of the runtime once per device; 256 without one).
inline int compute_units()
{
    static std::atomic<int> cached[64];  // zero-initialised; concurrent first calls store the same value
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// x / d from ceil(2^32 / d), exact for x d < 2^32; 0 stands for d = 1.  An integer division is some 25 dependent instructions, and six
// of them stood in front of a workgroup's first load: with these, and the arguments' lines asked for together, 24 heads, 2048 tokens
// (two kernels) 20.3 -> 19.8 us, 1200 tokens 14.9 -> 14.2, 300 tokens of 256 heads 12.6 -> 11.8, 1531 of 128 behind the convolution
// 46.2 -> 45.8.
inline uint32_t reciprocal(uint32_t d) { return d > 1 ? (uint32_t)((((uint64_t)1 << 32) + d - 1) / d) : 0u; }
__device__ __forceinline__ int quotient(int x, uint32_t inv)
{
    const int q = (int)(((uint64_t)(uint32_t)x * inv) >> 32);
    return inv ? q : x;
}
// ... of any 0 <= x < 2^31, for one instruction more: from ceil(2^(31 + k) / d), 2^(k - 1) < d <= 2^k, which fits 32 bits; rounded up
// it makes the quotient less than 2^-k <= 1 / d too large.  inv = 0 stands for d = 1.
struct Divisor {
    uint32_t inv;
    int32_t shift;
};
inline Divisor divisor(uint32_t d)
{
    if (d < 2) return {0u, 0};
    int k = 1;
    while (((uint64_t)1 << k) < d) ++k;
    return {(uint32_t)((((uint64_t)1 << (31 + k)) + d - 1) / d), k - 1};
}
__device__ __forceinline__ int quotient(int x, const Divisor &d)
{
    const int q = (int)((uint32_t)(((uint64_t)(uint32_t)x * d.inv) >> 32) >> d.shift);
    return d.inv ? q : x;
}

// Lets a kernel that takes dynamic LDS only use all of it.  The attribute belongs to the (kernel, device) pair and does
// not change, so the runtime is asked once for each and not on every launch.
template <auto Kernel>
hipError_t allow_full_lds()
{
    static std::atomic<uint64_t> done{0};  // one bit per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && (done.load(std::memory_order_relaxed) >> dev & 1u)) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kLdsPerCu);
    if (e == hipSuccess && dev >= 0 && dev < 64) done.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    return e;
}

// Device pointers of one call, shared by all kernels.
struct SsdArgs {
    quamba_ssd_shape_t s;
    const float *x_scales;
    const int32_t *head_cluster_end;
    const int32_t *chan_cluster_end;
    const float *B_scales;
    const float *C_scales;
    const int8_t *x;
    const int8_t *B;
    const int8_t *C;
    const float *dt;
    const float *A;
    const float *D;            // may be null
    const float *init_state;   // may be null (prefill)
    float *state;              // decode: in/out; prefill: final state or null
    uint16_t *y;               // fp16 bits
    // optional 8-bit side inputs (quamba_ssd_gate_t); all null / zero when absent
    const int8_t *z;           // gate codes, laid out like x
    float z_scale;
    const int8_t *dt_q;        // codes of the step size's pre-activation, laid out like dt (dt is then unused)
    float dt_scale;
    const float *dt_bias;      // [nheads] or null
    // Sequence split of the chunked prefill (matrix-core kernels only; nseg == 1: none).  The sequence is cut into nseg
    // segments of seg_chunks 128-token chunks (the last takes the rest).  A first kernel walks segments 0 .. nseg-2
    // without producing outputs and leaves, per segment, the state it ends with when started from zero (segment 0:
    // from init_state) and the sum of dt*A*log2(e) over its tokens; the prefill kernel then gives every segment its
    // own workgroups, which start from the combination of those.
    int32_t nseg;
    int32_t seg_chunks;
    float *seg_state;          // [nseg-1][batch*nheads][headdim * d_state], in the kernel's accumulator units and order
    float *seg_decay;          // [nseg-1][batch*nheads]
    int32_t pace_first;        // matrix-core prefill: first workgroup id of the second dispatch round when the two
                               // workgroups of a compute unit are to be kept at the same pace (see the kernel), else
                               // INT_MAX
    // Reciprocals for the kernels of short batches (quotient), whose start counts and that have at most a few thousand workgroups, and what they divide
    uint32_t inv_wgs_per_seg, inv_heads_per_group, inv_groups, inv_heads;
    int32_t heads_per_group, wgs_per_seg;
};

static_assert(sizeof(SsdArgs) == 248 && offsetof(SsdArgs, z) == 152 && offsetof(SsdArgs, pace_first) == 216, "tests/test_gpu_prefill.py repeats the layout");

// Plan of the matrix-core prefill for a shape on the current device: segments of the sequence split (1 = no split), chunks per
// segment, whether every head is cut into two workgroups of 32 channels each, and whether the workgroups are the wide
// kernel's.  It depends on what the call has besides x, B and C: the two-term state update, gate codes, step-size codes.
struct PrefillOperands {
    bool state, gate, dt_codes;
};
struct PrefillPlan {
    int nseg;
    int seg_chunks;
    bool channel_split;
    bool wide;
};
PrefillPlan prefill_mfma_plan(const quamba_ssd_shape_t &s, const PrefillOperands &with);
size_t prefill_mfma_workspace_bytes(const quamba_ssd_shape_t &s);

// Step size of (token or sequence) index idx of head h: the caller's fp32 dt, or softplus(s_dt * code + bias[h])
// (Section 3.2: Delta = softplus(F(x)) with the bias) when the pre-activation comes as int8 codes.
__device__ __forceinline__ float step_size_of_code(const SsdArgs &a, float code, int h)
{
    const float v = a.dt_scale * code + (a.dt_bias ? a.dt_bias[h] : 0.0f);
    return fmaxf(v, 0.0f) + log1pf(expf(-fabsf(v)));  // log(1 + exp(v)) without overflow
}
__device__ __forceinline__ float step_size(const SsdArgs &a, size_t idx, int h)
{
    return a.dt_q ? step_size_of_code(a, (float)a.dt_q[idx], h) : a.dt[idx];
}

// SiLU(z) = z / (1 + exp(-z)) of a gate code (Section 3.2: the optional branch z multiplies the SSM output).
__device__ __forceinline__ float silu_of_code(float z_scale, int code)
{
    const float z = z_scale * (float)code;
    return z * __frcp_rn(1.0f + __expf(-z));
}

// Index of the (group, head cluster, channel range) cell of channel position p of head h in the cluster boundary
// tables (Section 4.1: m x n cells per group).  The cluster index is the number of boundaries at or below the
// position, so all boundary loads are independent (three dependent memory round trips in total instead of one per
// boundary).
__device__ __forceinline__ int cell_lookup(const SsdArgs &a, int h, int p, int *first_cell_of_head = nullptr)
{
    const int hpg = a.s.nheads / a.s.ngroups;
    const int g = h / hpg, hl = h - g * hpg;
    const int m = a.s.n_head_clusters, n = a.s.n_chan_clusters;
    int i = 0;
    for (int k = 0; k < m - 1; ++k) i += hl >= a.head_cluster_end[g * m + k] ? 1 : 0;
    const int base = (g * m + i) * n;  // the head cluster's n cells are base .. base + n - 1
    if (first_cell_of_head) *first_cell_of_head = base;
    int j = 0;
    for (int k = 0; k < n - 1; ++k) j += p >= a.chan_cluster_end[base + k] ? 1 : 0;
    return base + j;
}

// First cell of head h's head cluster: the number of cluster ends at or below the head.  Up to 4 clusters are loaded at once
// (the last end is the group's head count, so reading it in place of the missing ones counts nothing).
__device__ __forceinline__ int head_cell_lookup(const SsdArgs &a, int g, int hl)  // head hl of group g
{
    const int m = a.s.n_head_clusters, n = a.s.n_chan_clusters;
    const int32_t *end = a.head_cluster_end + g * m;
    int i = 0;
    if (m <= 4) {
        const int e0 = end[0], e1 = end[min(1, m - 1)], e2 = end[min(2, m - 1)];
        i = (hl >= e0 ? 1 : 0) + (hl >= e1 ? 1 : 0) + (hl >= e2 ? 1 : 0);
        i = min(i, m - 1);
    } else {
        for (int k = 0; k < m - 1; ++k) i += hl >= end[k] ? 1 : 0;
    }
    return (g * m + i) * n;
}
__device__ __forceinline__ int head_cell_lookup(const SsdArgs &a, int h)
{
    const int hpg = a.s.nheads / a.s.ngroups, g = h / hpg;
    return head_cell_lookup(a, g, h - g * hpg);
}

// The channel ranges of a head cluster with up to 4 of them, in registers: ends of the first three and the four scales,
// loaded together (a missing range repeats the last one, whose end no position reaches).
struct Ranges4 {
    int e0, e1, e2;
    float s0, s1, s2, s3;
    __device__ __forceinline__ Ranges4(const SsdArgs &a, int base)
    {
        const int n = a.s.n_chan_clusters;
        const int k1 = base + min(1, n - 1), k2 = base + min(2, n - 1), k3 = base + min(3, n - 1);
        e0 = a.chan_cluster_end[base];
        e1 = a.chan_cluster_end[k1];
        e2 = a.chan_cluster_end[k2];
        s0 = a.x_scales[base];
        s1 = a.x_scales[k1];
        s2 = a.x_scales[k2];
        s3 = a.x_scales[k3];
    }
    // (conversions to values: a choice between members would be a choice between addresses, in memory)
    __device__ __forceinline__ float pick(int p) const
    {
        const float lo = p >= e0 ? float(s1) : float(s0), hi = p >= e2 ? float(s3) : float(s2);
        return p >= e1 ? float(hi) : float(lo);
    }
};

// Scale of channel position p of head h (Section 4.1: one scale per cell): the scale behind the last boundary at or below
// p.  The boundaries and the scales of the head cluster are loaded together, so two memory round trips stand in front
// of the result (the cell's index first would be a third).
__device__ __forceinline__ float x_scale_lookup(const SsdArgs &a, int h, int p)
{
    const int hpg = a.s.nheads / a.s.ngroups;
    const int g = h / hpg, hl = h - g * hpg;
    const int m = a.s.n_head_clusters, n = a.s.n_chan_clusters;
    int i = 0;
    for (int k = 0; k < m - 1; ++k) i += hl >= a.head_cluster_end[g * m + k] ? 1 : 0;
    const int base = (g * m + i) * n;
    float scale = a.x_scales[base];
    for (int k = 0; k < n - 1; ++k) {
        const int end = a.chan_cluster_end[base + k];
        const float next = a.x_scales[base + k + 1];
        scale = p >= end ? next : scale;
    }
    return scale;
}

// The same with the loads of the two steps unrolled, for calls that wait for the result: loops of unknown length are not
// unrolled into loads that fly together.
__device__ __forceinline__ float x_scale_lookup_wide(const SsdArgs &a, int h, int p)
{
    if (a.s.n_chan_clusters > 4) return x_scale_lookup(a, h, p);
    return Ranges4(a, head_cell_lookup(a, h)).pick(p);
}

// fp32 -> fp16 bits, round to nearest even.
__device__ __forceinline__ uint16_t f32_to_f16_bits(float v)
{
    const _Float16 h = (_Float16)v;
    return __builtin_bit_cast(uint16_t, h);
}

__device__ __forceinline__ float from_bits(uint32_t u) { return __builtin_bit_cast(float, u); }

// exp(z) for z <= 0 as separately rounded fp32 steps: t = z log2(e), k = rint(t), f = t - k in [-1/2, 1/2],
// 2^f = sum_i ((ln 2)^i / i!) f^i (i = 7..0, Horner, multiply then add), result 2^f 2^k; t < -125 gives 0 so that
// no result is subnormal.  Constants are the fp32 roundings of log2(e) and of the Taylor coefficients.  Used where an
// integer code depends on the result, so that it is the same fixed sequence of roundings on every machine.
__device__ __forceinline__ float exp_steps(float z)
{
#pragma clang fp contract(off)
    const float t = z * from_bits(0x3FB8AA3Bu);
    const float k = __builtin_rintf(t);
    const float f = t - k;
    float p = from_bits(0x377FE5FEu);
    p = p * f; p = p + from_bits(0x39218489u);
    p = p * f; p = p + from_bits(0x3AAEC3FFu);
    p = p * f; p = p + from_bits(0x3C1D955Bu);
    p = p * f; p = p + from_bits(0x3D635847u);
    p = p * f; p = p + from_bits(0x3E75FDF0u);
    p = p * f; p = p + from_bits(0x3F317218u);
    p = p * f; p = p + 1.0f;
    return t < -125.0f ? 0.0f : __builtin_ldexpf(p, (int)k);
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// Sum over groups of LANES consecutive lanes (LANES a power of two <= 64); every lane of a group gets the sum.
// Steps inside a row of 16 lanes are data-parallel-primitive moves fused into the adds (no LDS traffic): swap
// inside pairs, swap pairs inside quads, mirror inside 8, mirror inside 16; the step across rows is one swizzle.
template <int LANES>
__device__ __forceinline__ float group_sum(float v)
{
    if (LANES >= 2) v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
    if (LANES >= 4) v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
    if (LANES >= 8) v += dpp_move<0x141>(v);  // row_half_mirror
    if (LANES >= 16) v += dpp_move<0x140>(v); // row_mirror
    if (LANES >= 32)  // lane ^ 16
        v += __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
    if (LANES >= 64) v += __shfl_xor(v, 32, 64);
    return v;
}

// Scans of h <- dec h + in over groups of LANES lanes with E consecutive tokens each: is h, the scan's state in front of each
// lane's tokens, what the recurrence gives?  The scan's products of decays do not give it where a number is not finite: an
// infinite state times a product that underflows, or a product that overflows times a state of zero, is no number,
// while step by step the state stays infinite, or zero.  The answer is the wave's.
__device__ __forceinline__ bool scan_is_finite(float h)
{
    return __builtin_expect(__builtin_amdgcn_ballot_w64(!(__builtin_fabsf(h) < __builtin_inff())) == 0, 1);
}

// The same for the lane's group of LANES lanes alone.
template <int LANES>
__device__ __forceinline__ bool group_is_finite(float h)
{
    const uint64_t wave = __builtin_amdgcn_ballot_w64(!(__builtin_fabsf(h) < __builtin_inff()));
    return LANES == 64 ? wave == 0 : (wave >> (__lane_id() & ~(LANES - 1)) & ((1ull << (LANES & 63)) - 1)) == 0;
}

// The state in front of each lane's tokens, the group's lanes taking their tokens one after the other from `carried`, the
// state in front of the first.
template <int LANES, int E>
__device__ __forceinline__ float walk_lanes(float carried, const float (&dec)[E], const float (&in)[E])
{
    const int lane = __lane_id();
    float mine = carried;
#pragma unroll 1
    for (int l = 0; l < LANES; ++l) {
        float e = carried;
#pragma unroll
        for (int i = 0; i < E; ++i) e = fmaf(dec[i], e, in[i]);
        mine = (lane & (LANES - 1)) == l ? carried : mine;
        carried = __shfl(e, (lane & ~(LANES - 1)) | l, 64);
    }
    return mine;
}

hipError_t launch_decode(const SsdArgs &a, hipStream_t stream);
// 8-bit cached state (Appendix E): the step on int8 codes in place, and the quantizer of an fp32 state (a.state)
hipError_t launch_decode_q8(const SsdArgs &a, const float *state_scales, int8_t *state_q, hipStream_t stream);
hipError_t launch_quantize_state(const SsdArgs &a, const float *state_scales, int8_t *state_q, hipStream_t stream);
size_t decode_q8_lds_bytes(const quamba_ssd_shape_t &s);
struct Q8Plan {    // launch shape of the step's vector kernel: nheads x shares workgroups
    int shares;    // parts of the batch
    int seqs;      // sequences per slice of a part; 0: the shape does not fit, the any-shape kernel takes it
    int resident;  // workgroups the device holds at once
};
Q8Plan decode_q8_plan(const quamba_ssd_shape_t &s, bool gated);
// Quantized Hadamard transform of rows of n = 2^k fp16 values (Section 4.2)
hipError_t launch_hadamard_quantize(const uint16_t *y, int64_t rows, int n, float s_y, int8_t *out, hipStream_t stream);
bool hadamard_order_supported(int n);  // 2^k, or 12 * 2^k / 20 * 2^k with k >= 2, up to 16384
// W8A8 causal convolution in front of the scan (4 taps, SiLU, Eq. 1 to the scan's operands)
struct ConvArgs {
    quamba_ssd_shape_t s;
    const float *x_scales;
    const int32_t *head_cluster_end;
    const int32_t *chan_cluster_end;
    const float *B_scales;
    const float *C_scales;
    const int8_t *in;         // [b, L, HP + 2 GN]
    const int8_t *weight;     // [HP + 2 GN, 4]
    const float *bias;        // [HP + 2 GN] or null
    float in_w_scale;
    const int8_t *state_in;   // [b, 3, HP + 2 GN] or null
    int8_t *state_out;        // same shape, or null
    int8_t *x_out, *B_out, *C_out;
    int seg;                  // tokens per workgroup (set by the launcher, as what follows)
    int heads_per_group;
    Divisor by_headdim, by_heads_per_group, by_d_state;
};
bool conv1d_takes_four_channels(const quamba_ssd_shape_t &s);  // to a thread, where the addresses are aligned
hipError_t launch_conv1d_q8(const ConvArgs &a, hipStream_t stream);
constexpr int kMaxGridY = 65535;                    // of a launch
constexpr int kConvMaxTokens = 32 * kMaxGridY;  // longest sequence of the convolution (segments of 32 tokens)
// Mamba1 selective scan: shape has nheads = ngroups = 1, headdim = channels; A is [channels, d_state]
// Which kernel takes a scan: by lanes per channel, or channels per workgroup, or mamba1_scan_halves_kernel, or the one for any shape
enum class Mamba1Form : int { any, lanes16, lanes32, lanes64, channels8, channels24, halves };
Mamba1Form mamba1_scan_form(const quamba_ssd_shape_t &s);
bool mamba1_scan_mixes(const quamba_ssd_shape_t &s);  // channels24: mamba1_scan_mixed_kernel
hipError_t launch_mamba1_scan(const SsdArgs &a, const float *A, const float *init, float *fin, hipStream_t stream);
hipError_t launch_mamba1_decode(const SsdArgs &a, const float *A, hipStream_t stream);
bool mamba1_scan_supports_any(const quamba_ssd_shape_t &s);
hipError_t launch_prefill_generic(const SsdArgs &a, hipStream_t stream);
bool prefill_mfma_supports(const quamba_ssd_shape_t &s);
hipError_t launch_prefill_mfma(const SsdArgs &a, void *workspace, hipStream_t stream);
// Launches whose last round of workgroups is shared (prefill_mfma.hip).  polls: how often a piece looks for the one in front of it
// before it does without; 0: the default; below 0: it does without.
bool prefill_mfma_shares_rounds(const quamba_ssd_shape_t &s);
// Calls without a workspace of their own use the library's scratch memory: not where they share rounds, nor up to 7 chunks, since such
// calls may run side by side.
bool prefill_mfma_takes_scratch(const quamba_ssd_shape_t &s);
hipError_t launch_prefill_shared(const SsdArgs &a, void *workspace, bool precise, int polls, hipStream_t stream);
hipError_t launch_prefill_wide(const SsdArgs &a, bool halves, bool precise, hipStream_t stream);
bool prefill_generic_supports(const quamba_ssd_shape_t &s);

}  // namespace quamba
