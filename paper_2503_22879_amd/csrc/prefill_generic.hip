// Shape-agnostic prefill: the recurrence of Eq. 2 in fp32, for the shapes the chunked MFMA kernel does not take (any
// headdim, d_state, seqlen and alignment) and as an on-device cross-check of it.
//
// A row of the state (one channel of one head) needs nothing of the other rows, and along the sequence the recurrence is a
// scan, so a workgroup takes 16 rows (4 in small launches) and tiles of 256 tokens: 16 lanes share a row, 16 consecutive tokens each.  The
// decay depends on the head and the token alone, so its products over the lanes' tokens and the scan's products of those
// are formed once per tile and serve every state; per state a lane then folds its 16 inputs into one value, four
// data-parallel-primitive steps carry it across the row's lanes, and the lane replays its tokens from the state in front
// of them while it adds to y: 4 multiply-adds per (token, state), no exponential.  What bounds it at the sizes it is for
// (small models) is the latency of that chain, not a unit.  One workgroup per head that walked the tokens one after the
// other took 5.4 us per token (8 heads of 64 channels, 16 states, 256 tokens: 1388 us, now 5.9 us).
#include <type_traits>

#include "quamba_internal.h"

namespace quamba {
namespace {

constexpr int kE = 16;             // tokens per lane
constexpr int kLanes = 16;         // lanes per row
constexpr int kTile = kE * kLanes; // tokens per tile
constexpr int kNG = 16;            // states staged at a time
// Floats from one (state, quarter) of the staged B or C to the next.  A pad of 16 puts the writes of 64 consecutive tokens on as many
// banks: where four lane groups share a row, a unit has at most two workgroups whatever they take.  With one lane group three share
// a unit, for which 16 more KB between them would leave no room (see launch_rows).
constexpr int b_pitch(int SG) { return 4 * kLanes + (SG == 4 ? 16 : 4); }
constexpr int kXPitch = kTile + 16;      // bytes from one row's codes to the next
constexpr int kYPitch = kTile + 2;       // halves from one row's outputs to the next
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float code_to_float(uint32_t w, int k) { return (float)(int)(int8_t)(w >> (8 * k)); }

// v of the lane STEP positions earlier in the row of 16 lanes, `edge` where there is none.
template <int STEP>
__device__ __forceinline__ float row_earlier(float edge, float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v),
                                                                 0x110 + STEP, 0xf, 0xf, false));
}

constexpr size_t kernel_lds_bytes(int N, int rows, int SG)
{
    return sizeof(float) * (2 * kNG * 4 * b_pitch(SG) + 2 * kTile + rows * (size_t)N) + rows * kXPitch + 2 * rows * kYPitch;
}

// WIDE: d_state is a multiple of 4 and B and C are 4-byte aligned (their codes are read 4 at a time).
// SG: groups of 16 lanes that share a row, each with every SG-th state.  1: a wave holds 4 rows.  4: a wave is one row, whose
// four sums meet at the end; four times the waves with a quarter of the chain, for launches that would leave the chip empty.
// ROWS: rows per workgroup.  4 (with SG = 4, one wave per SIMD) puts a small launch on four times the compute units: 16 waves on
// one unit issue 9400 cycles of vector instructions, 3.9 of 7.9 us at 8 heads of 64 channels, 16 states, 256 tokens (now 5.9);
// a lane then has the registers to take all its states of a group side by side (four chains of multiply-adds instead of one), and
// of its 10000 cycles 2400 go by until the arguments are there, 2000 until the tile's loads are, 1200 in the staging and 2900
// in the states.
// WAVES: of a SIMD, for which registers are kept free (1: the compiler takes what it likes).
template <bool WIDE, int SG, int ROWS, int WAVES>
__global__ __launch_bounds__(ROWS * kLanes * SG, WAVES) void prefill_generic_kernel(SsdArgs a, int x_vec, int y_vec)
{
    constexpr int kRows = ROWS, kThreads = ROWS * kLanes * SG, kBPitch = b_pitch(SG);
    static_assert(kThreads >= kTile, "a thread for every (row, lane group, lane), and for every token of the tile");
    typedef uint32_t xcodes __attribute__((ext_vector_type(ROWS / 4)));
    extern __shared__ f32x4 lds4[];
    float *s_B = reinterpret_cast<float *>(lds4);  // [kNG][4][kBPitch]: state, quarter of a lane's tokens, lane x 4 tokens
    float *s_C = s_B + kNG * 4 * kBPitch;          // the same, times s_C
    float *s_dec = s_C + kNG * 4 * kBPitch;        // [kTile] exp(dt A)
    float *s_dtB = s_dec + kTile;                  // [kTile] dt s_B
    unsigned char *s_x = reinterpret_cast<unsigned char *>(s_dtB + kTile);  // [kRows][kXPitch] codes
    uint16_t *s_y = reinterpret_cast<uint16_t *>(s_x + kRows * kXPitch);    // [kRows][kYPitch]
    float *s_H = reinterpret_cast<float *>(s_y + kRows * kYPitch);          // [kRows][N] state in front of the tile

    const int L = a.s.seqlen, H = a.s.nheads, P = a.s.headdim, N = a.s.d_state, G = a.s.ngroups;
    const int bh = blockIdx.x, p0 = blockIdx.y * kRows;
    const int b = bh / H, h = bh - b * H, g = h / (H / G);
    const int rows = min(kRows, P - p0);
    const int tid = threadIdx.x, row = tid / (kLanes * SG), grp = (tid / kLanes) & (SG - 1), sub = tid & (kLanes - 1);
    const bool own = row < rows;
    const float Ah = a.A[h], Dh = a.D ? a.D[h] : 0.0f;
    const float sB = a.B_scales[g], sC = a.C_scales[g];
    const size_t st0 = ((size_t)bh * P + p0) * N;  // the workgroup's rows of the states

    float sx = 0.0f;
    auto look_up = [&]() {
        for (int e = tid; e < rows * N; e += kThreads) s_H[e] = a.init_state ? a.init_state[st0 + e] : 0.0f;
        sx = ROWS == 4 ? x_scale_lookup_wide(a, h, p0 + min(row, rows - 1)) : x_scale_lookup(a, h, p0 + min(row, rows - 1));
    };
    if (ROWS == 16) look_up();
    for (int t0 = 0; t0 < L; t0 += kTile) {
        const int nt = min(kTile, L - t0);
        const size_t tok0 = (size_t)b * L + t0;
        // B and C of a group of states, transposed: state-major, fp32.  A thread takes 4 states at a time of one token; all of its
        // loads are on their way before the first is used.
        constexpr int kItems = kTile * kNG / 4 / kThreads;  // such quads per thread and group
        const int t_bc = tid & (kTile - 1), quad0 = tid / kTile;
        uint32_t bw[kItems], cw[kItems];
        auto load_bc = [&](int n0, int ns) {
            if (!WIDE) return;
            const size_t off = ((tok0 + min(t_bc, nt - 1)) * G + g) * N + n0;
#pragma unroll
            for (int i = 0; i < kItems; ++i) {
                const int n = min(4 * (quad0 * kItems + i), ns - 4);
                bw[i] = *reinterpret_cast<const uint32_t *>(a.B + off + n);
                cw[i] = *reinterpret_cast<const uint32_t *>(a.C + off + n);
            }
        };
        auto put_bc = [&](int n, int t, float bv, float cv) {
            const int at = (n * 4 + ((t >> 2) & 3)) * kBPitch + 4 * (t >> 4) + (t & 3);
            s_B[at] = bv;
            s_C[at] = sC * cv;
        };
        auto stage_bc = [&](int n0, int ns) {
            if (WIDE) {
#pragma unroll
                for (int i = 0; i < kItems; ++i) {
                    const int n = 4 * (quad0 * kItems + i);
                    if (n >= ns) break;
                    if (t_bc >= nt) bw[i] = cw[i] = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) put_bc(n + k, t_bc, code_to_float(bw[i], k), code_to_float(cw[i], k));
                }
            } else {
                for (int e = tid; e < kTile * ns; e += kThreads) {
                    const int t = e / ns, n = e - t * ns;
                    float bv = 0.0f, cv = 0.0f;
                    if (t < nt) {
                        const size_t off = ((tok0 + t) * G + g) * N + n0 + n;
                        bv = (float)a.B[off];
                        cv = (float)a.C[off];
                    }
                    put_bc(n, t, bv, cv);
                }
            }
        };
        // thread = token: decay, step size, and the token's codes of the 16 rows.  Tokens past the end are identity
        // steps: decay 1, input 0.
        float dec_t = 1.0f, dtB_t = 0.0f;
        xcodes xq = (xcodes)(0u);
        const size_t dt_at = (tok0 + min(tid, nt - 1)) * H + h;
        const float dt_raw = a.dt_q ? (float)a.dt_q[dt_at] : a.dt[dt_at];
        load_bc(0, min(kNG, N));
        if (tid < nt) {  // nt <= kTile
            const int8_t *xp = a.x + ((tok0 + tid) * H + h) * P + p0;
            if (x_vec) {
                xq = *reinterpret_cast<const xcodes *>(xp);
            } else {
#pragma unroll
                for (int r = 0; r < kRows; ++r)
                    xq[r >> 2] |= (uint32_t)(uint8_t)xp[min(r, rows - 1)] << (8 * (r & 3));
            }
        }
        if (ROWS == 4 && t0 == 0) look_up();  // behind the first tile's loads: the look-ups wait for one another
        if (tid < nt) {
            const float dt = a.dt_q ? step_size_of_code(a, dt_raw, h) : dt_raw;
            dec_t = expf(dt * Ah);
            dtB_t = dt * sB;
        }
        stage_bc(0, min(kNG, N));
        if (tid < kTile) {
            s_dec[tid] = dec_t;
            s_dtB[tid] = dtB_t;
#pragma unroll
            for (int r = 0; r < kRows; ++r) s_x[r * kXPitch + tid] = (unsigned char)(xq[r >> 2] >> (8 * (r & 3)));
        }
        __syncthreads();

        // thread = (row, lane): decays, inputs and the start of the sums of its 16 tokens
        float dec[kE], u[kE], y[kE];
        float Pl[4];  // products of the decays over the lane's tokens and, after each step of the scan, its predecessors'
        {
            const u32x4 xc = *reinterpret_cast<const u32x4 *>(s_x + row * kXPitch + kE * sub);
            float prod = 1.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 d4 = *reinterpret_cast<const f32x4 *>(s_dec + kE * sub + 4 * q);
                const f32x4 b4 = *reinterpret_cast<const f32x4 *>(s_dtB + kE * sub + 4 * q);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = 4 * q + k;
                    const float xv = sx * code_to_float(xc[q], k);
                    dec[i] = d4[k];
                    u[i] = b4[k] * xv;
                    y[i] = SG == 1 || grp == 0 ? Dh * xv : 0.0f;
                    prod *= d4[k];
                }
            }
            Pl[0] = prod;
        }
        Pl[1] = Pl[0] * row_earlier<1>(1.0f, Pl[0]);
        Pl[2] = Pl[1] * row_earlier<2>(1.0f, Pl[1]);
        Pl[3] = Pl[2] * row_earlier<4>(1.0f, Pl[2]);
        const float Pin = Pl[3] * row_earlier<8>(1.0f, Pl[3]);  // over all tokens up to the lane's last
        const float Pex = row_earlier<1>(1.0f, Pin);            // in front of its first

        const int last = (nt - 1) / kE;  // the lane with the tile's last token: its replay ends with the state to carry on

        for (int n0 = 0; n0 < N; n0 += kNG) {
            const int ns = min(kNG, N - n0);
            if (n0) {  // the first group is staged with the tile's tokens
                load_bc(n0, ns);
                __syncthreads();
                stage_bc(n0, ns);
                __syncthreads();
            }
            // K states at a time, n and the following ones of the lane group: their chains run side by side
            auto states = [&](int n, auto count) {
                constexpr int K = decltype(count)::value;
                float in[K][kE], Hc[K], hh[K];
                bool finite = true;
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    Hc[j] = own ? s_H[row * N + n0 + n + j * SG] : 0.0f;
                    float hv = 0.0f;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 Bv = *reinterpret_cast<const f32x4 *>(s_B + ((n + j * SG) * 4 + q) * kBPitch + 4 * sub);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            in[j][4 * q + k] = u[4 * q + k] * Bv[k];
                            hv = fmaf(dec[4 * q + k], hv, in[j][4 * q + k]);
                        }
                    }
                    hv = fmaf(row_earlier<1>(0.0f, hv), Pl[0], hv);
                    hv = fmaf(row_earlier<2>(0.0f, hv), Pl[1], hv);
                    hv = fmaf(row_earlier<4>(0.0f, hv), Pl[2], hv);
                    hv = fmaf(row_earlier<8>(0.0f, hv), Pl[3], hv);
                    hh[j] = fmaf(Pex, Hc[j], row_earlier<1>(0.0f, hv));
                }
#pragma unroll
                for (int j = 0; j < K; ++j) finite = scan_is_finite(hh[j]) && finite;
                if (!finite) {
#pragma unroll
                    for (int j = 0; j < K; ++j) hh[j] = walk_lanes<kLanes>(Hc[j], dec, in[j]);
                }
#pragma unroll
                for (int j = 0; j < K; ++j) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 Cv = *reinterpret_cast<const f32x4 *>(s_C + ((n + j * SG) * 4 + q) * kBPitch + 4 * sub);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            hh[j] = fmaf(dec[4 * q + k], hh[j], in[j][4 * q + k]);
                            y[4 * q + k] = fmaf(Cv[k], hh[j], y[4 * q + k]);
                        }
                    }
                }
                // stored last: the compiler keeps LDS reads behind LDS writes
#pragma unroll
                for (int j = 0; j < K; ++j)
                    if (own && sub == last) s_H[row * N + n0 + n + j * SG] = hh[j];
            };
            int n = grp;
            // (two at a time take 160 registers, which 16 waves do not have)
            constexpr int kSide = SG == 1 ? 2 : ROWS == 4 ? 4 : 1;
            if (kSide > 1)
                for (; n + (kSide - 1) * SG < ns; n += kSide * SG) states(n, std::integral_constant<int, kSide>{});
            for (; n < ns; n += SG) states(n, std::integral_constant<int, 1>{});
        }
        // outputs: the groups' sums of a row meet (two exchanges that leave a group with 4 of the 16 tokens), then through
        // LDS to (token, row) order
        constexpr int kOut = kE / SG;  // tokens a lane puts out, from 4 grp on
        if (SG == 4) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {  // rows of 16 lanes 0, 1 keep token j, rows 2, 3 token j + 8
                const auto w = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, y[j]),
                                                                __builtin_bit_cast(uint32_t, y[j + 8]), false, false);
                y[j] = from_bits(w[0]) + from_bits(w[1]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // of those, even rows keep token j, odd rows j + 4
                const auto w = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, y[j]),
                                                                __builtin_bit_cast(uint32_t, y[j + 4]), false, false);
                y[j] = from_bits(w[0]) + from_bits(w[1]);
            }
        }
#pragma unroll
        for (int i = 0; i < kOut; ++i) {
            const int t = kE * sub + 4 * grp + i;
            float v = y[i];
            if (a.z)  // y * SiLU(z), Section 3.2
                v *= silu_of_code(a.z_scale, a.z[((tok0 + min(t, nt - 1)) * H + h) * P + p0 + min(row, rows - 1)]);
            s_y[row * kYPitch + t] = f32_to_f16_bits(v);
        }
        __syncthreads();
        if (tid < nt) {
            uint16_t *yp = a.y + ((tok0 + tid) * H + h) * P + p0;
            if (y_vec) {
                xcodes o[2];
#pragma unroll
                for (int r = 0; r < kRows; r += 2)
                    o[r / (kRows / 2)][(r / 2) % (kRows / 4)] =
                        (uint32_t)s_y[r * kYPitch + tid] | ((uint32_t)s_y[(r + 1) * kYPitch + tid] << 16);
                reinterpret_cast<xcodes *>(yp)[0] = o[0];
                reinterpret_cast<xcodes *>(yp)[1] = o[1];
            } else {
                for (int r = 0; r < rows; ++r) yp[r] = s_y[r * kYPitch + tid];
            }
        }
    }
    if (a.state) {
        __syncthreads();
        for (int e = tid; e < rows * N; e += kThreads) a.state[st0 + e] = s_H[e];
    }
}

template <bool WIDE, int SG, int ROWS, int WAVES>
hipError_t launch(const SsdArgs &a, hipStream_t stream)
{
    const hipError_t e = allow_full_lds<prefill_generic_kernel<WIDE, SG, ROWS, WAVES>>();
    if (e != hipSuccess) return e;
    auto aligned = [](const void *p, size_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
    const int whole = a.s.headdim % ROWS == 0;  // every row block is complete and starts at a multiple of ROWS codes
    const dim3 grid((unsigned)(a.s.batch * a.s.nheads), (unsigned)((a.s.headdim + ROWS - 1) / ROWS));
    hipLaunchKernelGGL((prefill_generic_kernel<WIDE, SG, ROWS, WAVES>), grid, dim3(ROWS * kLanes * SG),
                       kernel_lds_bytes(a.s.d_state, ROWS, SG), stream, a, whole && aligned(a.x, ROWS), whole && aligned(a.y, ROWS));
    return hipGetLastError();
}

static_assert(3 * kernel_lds_bytes(80, 16, 1) <= kLdsPerCu, "three workgroups of 16 rows per compute unit");

template <bool WIDE>
hipError_t launch_rows(const SsdArgs &a, hipStream_t stream)
{
    // Blocks of 16 rows.  Up to one per compute unit: four lane groups per row (16 waves) instead of one (4 waves).  Up to one per
    // two units: blocks of 4 rows (4 waves), of which a unit holds two with the registers they take (8 heads of 64 channels, 16
    // states, 256 tokens, 16 / 4 rows: batch 1 7.8 / 5.9 us, 4 8.3 / 7.4, 5 8.4 / 11.4; 24 heads, 64 states, 1000 tokens 53.9 / 45.4).
    // Codes that are read one at a time cost the four-fold staging more than the waves gain (10 states, 200 tokens 7.7 / 9.5).
    // Above two per unit a third one has to fit, in 168 registers and 51 KB (16 states; 8 heads of 64 channels, 256 tokens, with 174
    // registers and 57 KB / so: batch 17 17.8 / 13.2 us, 64 42.1 / 36.3; 17 of 64 states 51.3 / 35.6).  Up to there 174 are the better
    // (batch 16 11.4 / 11.8).
    const int64_t blocks = (int64_t)a.s.batch * a.s.nheads * ((a.s.headdim + 15) / 16);
    if (blocks > 2 * (int64_t)compute_units()) return launch<WIDE, 1, 16, 3>(a, stream);
    if (blocks > compute_units()) return launch<WIDE, 1, 16, WIDE ? 1 : 3>(a, stream);
    if constexpr (WIDE)
        if (2 * blocks <= compute_units()) return launch<WIDE, 4, 4, 1>(a, stream);
    return launch<WIDE, 4, 16, 1>(a, stream);
}

}  // namespace

// The shapes the entry points take: headdim * d_state bounded by the LDS of a compute unit (the documented limit of this
// path, which the kernel's own need stays below).
bool prefill_generic_supports(const quamba_ssd_shape_t &s)
{
    const size_t P = (size_t)s.headdim, N = (size_t)s.d_state;
    return sizeof(float) * (P * N + 33 * P + 32 * N + 16) <= kLdsPerCu && kernel_lds_bytes(s.d_state, 16, 4) <= kLdsPerCu;
}

hipError_t launch_prefill_generic(const SsdArgs &a, hipStream_t stream)
{
    const bool wide = a.s.d_state % 4 == 0 && reinterpret_cast<uintptr_t>(a.B) % 4 == 0 && reinterpret_cast<uintptr_t>(a.C) % 4 == 0;
    return wide ? launch_rows<true>(a, stream) : launch_rows<false>(a, stream);
}

}  // namespace quamba
