// Single-token decode of the 8-bit SSD: one step of Eq. 2 on the persistent fp32 state, in place.
//
// The step is a pure stream over the state (read 4 B + write 4 B per element, 3 FMAs), so the kernel is built
// around HBM: one workgroup per (sequence, head), every lane owns 16-byte pieces of state rows, all of a lane's
// loads are issued before any arithmetic, the d_state reduction of y stays in registers (cross-lane adds), and
// the de-quantized per-row input x is staged through a few hundred bytes of LDS by each wave for its own rows.
#include "quamba_internal.h"

namespace quamba {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// De-quantized x of this head into LDS: xv[p] = s_x(h,p) * xq[p] (inverse of Eq. 1 with the m x n table).
__device__ __forceinline__ void stage_x(const SsdArgs &a, int bh, int h, float *xv)
{
    const int P = a.s.headdim;
    for (int p = threadIdx.x; p < P; p += kThreads)
        xv[p] = x_scale_lookup(a, h, p) * (float)a.x[(size_t)bh * P + p];
}

// Fast path: d_state = N (multiple of 4, N/4 a power of two <= 64).  A row of N floats is covered by N/4 lanes with
// one float4 each; a wave covers 64/(N/4) rows per load instruction and keeps ROWS such instructions in flight.
// FULL: headdim is a multiple of the rows one pass of the workgroup covers, so no row needs clamping or masking and
// the row addresses are one base plus compile-time offsets.
// ONE: a workgroup takes one pass (blockIdx.y says which) instead of the whole head.  At small batches the step is a chain
// of memory round trips, so the passes run side by side, everything a row needs besides its state (scale, x, gate) is
// requested in front of the state, the state in front of everything that waits, and nothing is loaded behind it (24 heads
// at batch 1: 7.5 -> 4.6 us).
template <int N, int ROWS, bool FULL, bool ONE>
__global__ __launch_bounds__(kThreads) void decode_vec_kernel(SsdArgs a)
{
    constexpr int LPR = N / 4;     // lanes per row
    constexpr int RPI = 64 / LPR;  // rows per wave-wide load
    constexpr int PASS = kWaves * RPI * ROWS;  // rows of a pass of the workgroup
    static_assert(RPI * ROWS <= 64, "one lane per row of a pass");
    extern __shared__ float lds[];
    const int P = a.s.headdim, H = a.s.nheads, G = a.s.ngroups;
    float *xv = lds;                   // [P], or [PASS]
    __shared__ float s_gate[ONE ? PASS : 1];

    const int bh = blockIdx.x;
    const int b = bh / H, h = bh - b * H, g = h / (H / G);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane % LPR, sub = lane / LPR;
    const int first = ONE ? (int)blockIdx.y * PASS : 0;
    const int p_begin = first + wave * RPI * ROWS;
    if (ONE && !FULL && p_begin >= P) return;

    float *st = a.state + (size_t)bh * P * N + 4 * j;
    f32x4 v[ROWS];
    // all of the lane's loads of a pass together, unconditionally (rows past the end re-read the last row and are not
    // stored)
    auto request_state = [&](int p0) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int p = FULL ? p0 + i * RPI + sub : min(p0 + i * RPI + sub, P - 1);
            v[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(st + (size_t)p * N));
        }
    };
    int8_t xq = 0, zq = 0;
    float sx = 0.0f;
    if (ONE) {  // one lane per row
        const int p = min(p_begin + min(lane, RPI * ROWS - 1), P - 1);
        xq = a.x[(size_t)bh * P + p];
        if (a.z) zq = a.z[(size_t)bh * P + p];
        sx = x_scale_lookup_wide(a, h, p);
        request_state(p_begin);
    }
    const float dt = step_size(a, bh, h);
    const float dA = expf(dt * a.A[h]);
    const float Dh = a.D ? a.D[h] : 0.0f;
    const float sB = a.B_scales[g] * dt, sC = a.C_scales[g];
    const char4 bq = *reinterpret_cast<const char4 *>(a.B + ((size_t)b * G + g) * N + 4 * j);
    const char4 cq = *reinterpret_cast<const char4 *>(a.C + ((size_t)b * G + g) * N + 4 * j);
    const float4 Bv = make_float4(sB * bq.x, sB * bq.y, sB * bq.z, sB * bq.w);  // dt * B_t (B-dot of Sec. 3.2)
    const float4 Cv = make_float4(sC * cq.x, sC * cq.y, sC * cq.z, sC * cq.w);

    for (int p0 = p_begin; p0 < (ONE ? p_begin + 1 : P); p0 += PASS) {
        if (!ONE) request_state(p0);
        // de-quantized x of the rows of this trip, staged by the wave for itself while its state loads are in
        // flight: no workgroup barrier, the waves never wait for each other (LDS accesses of one wave stay in order)
        if (ONE) {
            if (lane < RPI * ROWS) {
                xv[p0 - first + lane] = sx * (float)xq;
                if (a.z) s_gate[p0 - first + lane] = silu_of_code(a.z_scale, zq);
            }
        } else {
            for (int r = lane; r < RPI * ROWS; r += 64) {
                const int p = p0 + r;
                if (FULL || p < P) xv[p] = x_scale_lookup(a, h, p) * (float)a.x[(size_t)bh * P + p];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float part[ROWS];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int p = FULL ? p0 + i * RPI + sub : min(p0 + i * RPI + sub, P - 1);
            const float x = xv[p - first];
            v[i].x = fmaf(dA, v[i].x, Bv.x * x);
            v[i].y = fmaf(dA, v[i].y, Bv.y * x);
            v[i].z = fmaf(dA, v[i].z, Bv.z * x);
            v[i].w = fmaf(dA, v[i].w, Bv.w * x);
            if (FULL || p0 + i * RPI + sub < P)
                __builtin_nontemporal_store(v[i], reinterpret_cast<f32x4 *>(st + (size_t)p * N));
            part[i] = fmaf(Cv.x, v[i].x, fmaf(Cv.y, v[i].y, fmaf(Cv.z, v[i].z, Cv.w * v[i].w)));
        }
#pragma unroll
        for (int i = 0; i < ROWS; ++i) part[i] = group_sum<LPR>(part[i]);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int p = p0 + i * RPI + sub;
            if (j == 0 && (FULL || p < P)) {
                float gate = 1.0f;  // y * SiLU(z)
                if (a.z) gate = ONE ? s_gate[p - first] : silu_of_code(a.z_scale, a.z[(size_t)bh * P + p]);
                a.y[(size_t)bh * P + p] = f32_to_f16_bits(fmaf(Dh, xv[p - first], part[i]) * gate);
            }
        }
    }
}

// Any d_state: one wave per row, lanes stride over the states.
__global__ __launch_bounds__(kThreads) void decode_any_kernel(SsdArgs a)
{
    extern __shared__ float lds[];
    const int P = a.s.headdim, H = a.s.nheads, G = a.s.ngroups, N = a.s.d_state;
    float *xv = lds;
    float *ys = lds + P;
    const int bh = blockIdx.x;
    const int b = bh / H, h = bh - b * H, g = h / (H / G);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    stage_x(a, bh, h, xv);
    __syncthreads();
    const float dt = step_size(a, bh, h);
    const float dA = expf(dt * a.A[h]);
    const float Dh = a.D ? a.D[h] : 0.0f;
    const float sB = a.B_scales[g] * dt, sC = a.C_scales[g];
    const int8_t *Bq = a.B + ((size_t)b * G + g) * N;
    const int8_t *Cq = a.C + ((size_t)b * G + g) * N;
    float *st = a.state + (size_t)bh * P * N;
    for (int p = wave; p < P; p += kWaves) {
        const float x = xv[p];
        float part = 0.0f;
        for (int n = lane; n < N; n += 64) {
            const float hn = fmaf(dA, st[(size_t)p * N + n], sB * (float)Bq[n] * x);
            st[(size_t)p * N + n] = hn;
            part = fmaf(sC * (float)Cq[n], hn, part);
        }
        part = group_sum<64>(part);
        if (lane == 0) ys[p] = fmaf(Dh, x, part);
    }
    __syncthreads();
    for (int p = threadIdx.x; p < P; p += kThreads) {
        const float gate = a.z ? silu_of_code(a.z_scale, a.z[(size_t)bh * P + p]) : 1.0f;  // y * SiLU(z)
        a.y[(size_t)bh * P + p] = f32_to_f16_bits(ys[p] * gate);
    }
}

template <int N>
hipError_t launch_vec(const SsdArgs &a, hipStream_t stream)
{
    constexpr int LPR = N / 4, RPI = 64 / LPR;
    constexpr int ROWS = (RPI * 4 * kWaves <= 64) ? 4 : (RPI <= 8 ? 2 : 1);  // rows per lane in flight per trip
    constexpr int PASS = kWaves * RPI * ROWS;  // rows of one pass of a workgroup
    const int P = a.s.headdim;
    // One pass per workgroup, except for the largest batches without a gate.  In a token's sequence of calls (convolution in
    // front, transform behind) the two orders meet between 140 and 190 workgroups per compute unit, within 1 % of each other
    // from 128 on (one pass / whole head, the three calls, 128 heads: batch 128 185.7 / 187.1 us, 192 277.8 / 277.4, 224
    // 323.6 / 322.4, 256 370.8 / 366.1; 80 heads: 224 202.7 / 203.5, 256 231.7 / 230.7, 400 364.2 / 358.2).  With a gate, whose
    // codes the other order reads behind the state, one pass is always ahead (128 heads, batch 256: 361.0 / 375.7); so it is
    // where the step is called alone, over and over (358.6 / 370.4), which no program does.
    const int64_t pairs = (int64_t)a.s.batch * a.s.nheads, passes = (P + PASS - 1) / PASS;
    if (a.z || pairs * passes <= 128 * (int64_t)compute_units()) {
        const dim3 grid((unsigned)pairs, (unsigned)passes);
        if (P % PASS == 0)
            hipLaunchKernelGGL((decode_vec_kernel<N, ROWS, true, true>), grid, dim3(kThreads), sizeof(float) * PASS, stream, a);
        else
            hipLaunchKernelGGL((decode_vec_kernel<N, ROWS, false, true>), grid, dim3(kThreads), sizeof(float) * PASS, stream, a);
    } else {
        const dim3 grid((unsigned)pairs);
        const size_t lds = sizeof(float) * (size_t)P;
        if (P % PASS == 0)
            hipLaunchKernelGGL((decode_vec_kernel<N, ROWS, true, false>), grid, dim3(kThreads), lds, stream, a);
        else
            hipLaunchKernelGGL((decode_vec_kernel<N, ROWS, false, false>), grid, dim3(kThreads), lds, stream, a);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(const SsdArgs &a, hipStream_t stream)
{
    const bool aligned = (reinterpret_cast<uintptr_t>(a.state) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(a.B) % 4 == 0) && (reinterpret_cast<uintptr_t>(a.C) % 4 == 0);
    if (aligned) {
        switch (a.s.d_state) {
            case 256: return launch_vec<256>(a, stream);
            case 128: return launch_vec<128>(a, stream);
            case 64: return launch_vec<64>(a, stream);
            case 32: return launch_vec<32>(a, stream);
            case 16: return launch_vec<16>(a, stream);
            default: break;
        }
    }
    const dim3 grid((unsigned)(a.s.batch * a.s.nheads));
    const size_t lds = sizeof(float) * 2 * (size_t)a.s.headdim;
    hipLaunchKernelGGL(decode_any_kernel, grid, dim3(kThreads), lds, stream, a);
    return hipGetLastError();
}

}  // namespace quamba
