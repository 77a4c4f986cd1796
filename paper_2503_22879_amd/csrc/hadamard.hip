// Quantized Hadamard transform of the SSD output (Section 4.2): out = Eq.1((1/s_y) H_n y) per row of n = 2^k values,
// the 8-bit input of the output projection whose weight carries the matching H_n offline.
//
// The transform is the radix-2 butterfly network with strides 1, 2, 4, ..., n/2 in this order, in fp32, every add and
// subtract rounded on its own (the codes are integers decided by these roundings, so the order is part of the
// definition; the header states it).  One workgroup per row at a time.  For n >= 1024 a thread keeps 32 values in
// registers and the network runs in three phases of up to 5 strides each, with the values redistributed through LDS
// in between so that the strides of a phase are register-local: phase A on 32 consecutive values (strides 1..16),
// phase B on values 32 apart (strides 32..512), phase C on values 1024 apart (strides 1024..n/2) for groups of
// consecutive values, so that the codes leave as dwords.  The row is read once (fp16, 64 contiguous bytes per thread)
// and written once (int8): 3 bytes of HBM traffic and 17 vector instructions (13 butterflies, a scale, a clamp, a
// rounding add; no packed fp32) per value.  At n = 8192 the vector ALU, the LDS exchanges and HBM each take 40-60 us
// when alone; a row's fp32 image (37 KB of LDS) limits a compute unit to 4 rows in flight, so they overlap only partly.
#include <atomic>

#include "quamba_internal.h"

#pragma clang fp contract(off)

namespace quamba {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32_u __attribute__((aligned(2)));  // the hardware stores dwords at any address
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr float kMagic = 12582912.0f;  // 1.5 * 2^23: adding it rounds to nearest even, the code is the sum's low byte

// Eq. 1 with the bounds of an 8-bit code for one value (the paths without packing).
__device__ __forceinline__ uint32_t code_byte(float r)
{
    const float c = __builtin_amdgcn_fmed3f(r, -128.0f, 127.0f);
    return __builtin_bit_cast(uint32_t, c + kMagic) & 0xffu;
}

// The same for K = 2 or 4 values packed into the low bytes of a dword: the rounding add writes its low byte straight
// into byte k of the result through the sub-dword destination select.
template <int K>
__device__ __forceinline__ uint32_t codes_packed(const float (&r)[4])
{
    float c[4];
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = __builtin_amdgcn_fmed3f(r[k], -128.0f, 127.0f);
    uint32_t out;
    asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD"
        : "=v"(out) : "v"(c[0]), "v"(kMagic));
    asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
        : "+v"(out) : "v"(c[1]), "v"(kMagic));
    if (K == 4) {
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
            : "+v"(out) : "v"(c[2]), "v"(kMagic));
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
            : "+v"(out) : "v"(c[3]), "v"(kMagic));
    }
    return out;
}

// The same without the sub-dword add, for the kernel that is bound by vector issue (see there): the sums' low bytes gathered by
// byte permutes.
template <int K>
__device__ __forceinline__ uint32_t codes_gathered(const float (&r)[4])
{
    uint32_t c[4];
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(r[k], -128.0f, 127.0f) + kMagic);
    const uint32_t lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u);
    if (K == 2) return lo;
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u), lo, 0x05040100u);
}

// In-register butterflies of one phase: v[e], e = 0..31, strides 1..2^(BITS-1) on the register index.
template <int BITS, int FIRST = 1>
__device__ __forceinline__ void butterflies(float (&v)[32])
{
#pragma unroll
    for (int h = FIRST; h < (1 << BITS); h <<= 1)
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if ((e & h) == 0) {
                const float a = v[e], b = v[e + h];
                v[e] = a + b;
                v[e + h] = a - b;
            }
}

// n = 2^LOGN, 10 <= LOGN <= 14, n/32 threads, as many workgroups as stay resident; each loops over rows
// blockIdx.x, blockIdx.x + gridDim.x, ... and loads its next row (16 registers of packed fp16) while it works on the
// current one, so the HBM latency of a row is hidden behind the arithmetic of the row before.  The loads are plain,
// not non-temporal: a lane's four 16-byte loads walk through one 64-byte sector, which has to stay in the vector cache
// between them (with non-temporal loads every one of the four fetched the sector again and the loads alone took 69 us
// instead of 39 at the 8B layer's size).
// Rows of fewer than 8192 values share a workgroup (8 rows of 1024, 4 of 2048, 2 of 4096), each with its own threads
// and its own piece of LDS, so that a workgroup always has 256 or 512 threads; the rows of a workgroup move through
// the phases together.
template <int LOGN>
constexpr int rows_per_workgroup() { return LOGN >= 13 ? 1 : 1 << (13 - LOGN); }

template <int LOGN>
__global__ __launch_bounds__((1 << (LOGN - 5)) * rows_per_workgroup<LOGN>()) void hadamard_quantize_kernel(
    const uint16_t *y, int8_t *out, int rows, float inv_s)
{
    constexpr int N = 1 << LOGN;
    constexpr int RPW = rows_per_workgroup<LOGN>(), T = N / 32;
    // phase C: a thread holds CONSEC consecutive values at NE places GS apart (4 x 8, n/8 apart; 2 x 16, 1024 apart for
    // n = 16384); the places' index bits that are strides >= 1024 still have their butterflies to come
    constexpr int NE = LOGN == 14 ? 16 : 8;
    constexpr int CONSEC = 32 / NE;
    constexpr int GS = N / NE;
    constexpr int CFIRST = LOGN >= 13 ? 1 : 1 << (13 - LOGN);  // first register stride of phase C that is a stride >= 1024
    extern __shared__ float lds_all[];  // per row 1152 floats per block of 1024 values
    const int t = threadIdx.x % T, rw = threadIdx.x / T;
    float *lds = lds_all + rw * (N / 1024) * 1152;
    const int t_lo = t & 31, t_hi = t >> 5;
    float v[32];
    u32x4 nx[4];
    const long long stride = (long long)gridDim.x * RPW;  // rows between two rounds of a thread

    long long r = (long long)blockIdx.x * RPW + rw;  // the launch has no more workgroups than groups of RPW rows
#pragma unroll
    for (int q = 0; q < 4; ++q) nx[q] = (u32x4){0, 0, 0, 0};
    if (r < rows) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(y + (size_t)r * N + 32 * t);
#pragma unroll
        for (int q = 0; q < 4; ++q) nx[q] = src[q];
    }
    // every thread of the workgroup makes the same number of rounds (the barriers below are the workgroup's); a thread
    // whose row lies past the end works on zeros and stores nothing
    for (long long r0 = (long long)blockIdx.x * RPW; r0 < rows; r0 += stride, r += stride) {
        // phase A: values 32 t + e;
        // stride 1 straight from the packed fp16 pairs: the mixed-precision fused multiply-add takes both halves of a
        // dword as fp16 sources, lo * 1.0 +- hi in fp32 with one rounding (conversion of fp16 to fp32 is exact, so
        // this is the fp32 add or subtract of the converted values)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t w = nx[q][i];
                asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(v[8 * q + 2 * i]) : "v"(w));
                asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]"
                    : "=v"(v[8 * q + 2 * i + 1]) : "v"(w));
            }
        if (r + stride < rows) {
            const u32x4 *src = reinterpret_cast<const u32x4 *>(y + (size_t)(r + stride) * N + 32 * t);
#pragma unroll
            for (int q = 0; q < 4; ++q) nx[q] = src[q];
        }
        butterflies<5, 2>(v);
        // Through LDS, transposed inside every block of 1024 values: value 32 a + k of the block (thread a's k-th
        // value) goes to 36 k + a, so that the 32 values the next phase needs in one thread (k fixed, a = 0..31) are
        // 32 consecutive floats, read 16 bytes at a time; the pitch of 36 floats keeps 16 lanes' 16-byte reads on
        // distinct banks, and the writes of consecutive threads are consecutive floats.
        {
            float *pa = lds + t_lo + 1152 * t_hi;
#pragma unroll
            for (int k = 0; k < 32; ++k) pa[36 * k] = v[k];
            __syncthreads();
            // phase B: values i = t_lo + 32 e + 1024 t_hi, e = 0..31
            const f32x4 *pb = reinterpret_cast<const f32x4 *>(lds + 36 * t_lo + 1152 * t_hi);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const f32x4 w = pb[q];
                v[4 * q] = w[0]; v[4 * q + 1] = w[1]; v[4 * q + 2] = w[2]; v[4 * q + 3] = w[3];
            }
        }
        butterflies<5>(v);
        __syncthreads();  // all reads of the transposed layout are done before the plain one overwrites it
        {
            float *pb = lds + t_lo + 1024 * t_hi;
#pragma unroll
            for (int e = 0; e < 32; ++e) pb[32 * e] = v[e];
        }
        __syncthreads();

        // phase C: CONSEC consecutive values at CONSEC t + GS e', e' = 0..NE-1; register index k * NE + e', so the
        // strides GS .. n/2 are its low bits, of which those below 1024 are already done
#pragma unroll
        for (int ep = 0; ep < NE; ++ep)
#pragma unroll
            for (int k = 0; k < CONSEC; ++k) v[k * NE + ep] = (lds + CONSEC * t)[k + GS * ep];
        butterflies<(LOGN == 14 ? 4 : 3), CFIRST>(v);

        // Eq. 1 and the store: CONSEC consecutive codes per e'
        int8_t *orow = out + (size_t)r * N + CONSEC * t;
#pragma unroll
        for (int ep = 0; ep < NE; ++ep) {
            if (r >= rows) break;
            if (CONSEC >= 4) {
#pragma unroll
                for (int k = 0; k < CONSEC; k += 4) {
                    const float sc[4] = {v[k * NE + ep] * inv_s, v[(k + 1) * NE + ep] * inv_s,
                                         v[(k + 2) * NE + ep] * inv_s, v[(k + 3) * NE + ep] * inv_s};
                    __builtin_nontemporal_store(codes_packed<4>(sc),
                                                reinterpret_cast<uint32_t *>(orow + GS * ep + k));
                }
            } else {
                const float sc[4] = {v[ep] * inv_s, v[NE + ep] * inv_s, 0.0f, 0.0f};
                *reinterpret_cast<uint16_t *>(orow + GS * ep) = (uint16_t)codes_packed<2>(sc);
            }
        }
        __syncthreads();  // phase C has read the row before the next row's phase A writes
    }
}

// Any power of two n <= 16384: the network stage by stage in LDS.
__global__ __launch_bounds__(256) void hadamard_quantize_small_kernel(const uint16_t *y, int8_t *out, int n, float inv_s)
{
    extern __shared__ float lds[];
    const size_t row = (size_t)blockIdx.x * n;
    for (int i = threadIdx.x; i < n; i += 256) {
        const _Float16 hv = __builtin_bit_cast(_Float16, y[row + i]);
        lds[i] = (float)hv;
    }
    __syncthreads();
    for (int h = 1; h < n; h <<= 1) {
        for (int k = threadIdx.x; k < n / 2; k += 256) {
            const int i = ((k & ~(h - 1)) << 1) | (k & (h - 1));  // k-th index with bit h clear
            const float a = lds[i], b = lds[i + h];
            lds[i] = a + b;
            lds[i + h] = a - b;
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < n; i += 256) out[row + i] = (int8_t)code_byte(lds[i] * inv_s);
}

// Orders m * 2^k, m = 12 or 20: H_n = H_m (x) H_{2^k} with H_m from Paley's first construction (q = m - 1 prime, 3 mod 4):
// H_m = I + S, S = [[0, 1^T], [-1, Q]], Q[i, j] = chi(i - j), chi the quadratic character mod q.  chi is a bit mask of
// the non-zero squares mod q, built at compile time.
constexpr uint32_t square_mask(int q)
{
    uint32_t mask = 0;
    for (int v = 1; v < q; ++v) mask |= 1u << ((v * v) % q);
    return mask;
}
template <int M>
constexpr float paley_sign(int a, int b)  // H_M[a][b] as +-1.0f
{
    constexpr int q = M - 1;
    if (a == 0 || a == b) return 1.0f;
    if (b == 0) return -1.0f;
    const int d = ((a - b) % q + q) % q;
    return (square_mask(q) >> d) & 1u ? 1.0f : -1.0f;
}

// One workgroup per row: the butterfly network inside every block of p = 2^k values stage by stage in LDS, then for
// every position j the M-point transform across the blocks, accumulated over the blocks in ascending order (the order
// the header states), Eq. 1, and the codes of 4 consecutive positions per store.
template <int M>
__global__ __launch_bounds__(256) void hadamard_quantize_mixed_kernel(const uint16_t *y, int8_t *out, int p, float inv_s,
                                                                     int out_aligned)
{
    extern __shared__ float lds[];
    const int n = M * p;
    const size_t row = (size_t)blockIdx.x * n;
    for (int i = threadIdx.x; i < n; i += 256) {
        const _Float16 hv = __builtin_bit_cast(_Float16, y[row + i]);
        lds[i] = (float)hv;
    }
    __syncthreads();
    for (int h = 1; h < p; h <<= 1) {
        for (int k = threadIdx.x; k < n / 2; k += 256) {
            const int i = ((k & ~(h - 1)) << 1) | (k & (h - 1));  // k-th index with bit h clear; h < p stays in a block
            const float a = lds[i], b = lds[i + h];
            lds[i] = a + b;
            lds[i + h] = a - b;
        }
        __syncthreads();
    }
    for (int j4 = threadIdx.x; j4 < p / 4; j4 += 256) {
        f32x4 t[M];
#pragma unroll
        for (int b = 0; b < M; ++b) t[b] = *reinterpret_cast<const f32x4 *>(lds + b * p + 4 * j4);
#pragma unroll
        for (int a = 0; a < M; ++a) {
            f32x4 acc = t[0] * paley_sign<M>(a, 0);
#pragma unroll
            for (int b = 1; b < M; ++b) acc = acc + t[b] * paley_sign<M>(a, b);
            const float sc[4] = {acc[0] * inv_s, acc[1] * inv_s, acc[2] * inv_s, acc[3] * inv_s};
            int8_t *dst = out + row + (size_t)a * p + 4 * j4;
            const uint32_t w = codes_packed<4>(sc);
            if (out_aligned) {
                *reinterpret_cast<uint32_t *>(dst) = w;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) dst[k] = (int8_t)(w >> (8 * k));
            }
        }
    }
}

// The words of the quad's neighbouring (lane ^ 1) or opposite (lane ^ 2) lanes, in one burst at raised wave priority, where it stays
// (two wait states between a vector instruction and a lane move of its result).
template <int STEP, int K>
__device__ __forceinline__ void swap_lanes(const uint32_t (&w)[K], uint32_t (&o)[K])
{
    static_assert(K == 3 || K == 5, "the rows of the 12- and 20-point sums, four to a word");
#define QUAMBA_MOVE(to, from, perm) "\n\tv_mov_b32_dpp %" #to ", %" #from " quad_perm:" perm " row_mask:0xf bank_mask:0xf"
#define QUAMBA_MOVE3(perm) QUAMBA_MOVE(0, 3, perm) QUAMBA_MOVE(1, 4, perm) QUAMBA_MOVE(2, 5, perm)
#define QUAMBA_MOVE5(perm) QUAMBA_MOVE(0, 5, perm) QUAMBA_MOVE(1, 6, perm) QUAMBA_MOVE(2, 7, perm) QUAMBA_MOVE(3, 8, perm) QUAMBA_MOVE(4, 9, perm)
#define QUAMBA_MOVE_ALL(perm)                                                                                             \
    if constexpr (K == 5)                                                                                                 \
        asm volatile("s_nop 1\n\ts_setprio 2" QUAMBA_MOVE5(perm)                                                          \
                     : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4])                                    \
                     : "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]));                                            \
    else                                                                                                                  \
        asm volatile("s_nop 1\n\ts_setprio 2" QUAMBA_MOVE3(perm)                                                          \
                     : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2])                                                              \
                     : "v"(w[0]), "v"(w[1]), "v"(w[2]));
    if constexpr (STEP == 0) {
        QUAMBA_MOVE_ALL("[1,0,3,2]")
    } else {
        QUAMBA_MOVE_ALL("[2,3,0,1]")
    }
#undef QUAMBA_MOVE_ALL
#undef QUAMBA_MOVE5
#undef QUAMBA_MOVE3
#undef QUAMBA_MOVE
}

// The same orders with the register-blocked phases of the power-of-two kernel (p = 2^LOGP values per block, 7 <= LOGP
// <= 10, 16-byte aligned rows): phase A, strides 1..16 on the 32 consecutive values a thread loads; exchange through
// LDS, transposed inside super-blocks of 1024 values like the power-of-two kernel's first exchange; phase B, strides
// 32..p/2 on values 32 apart (a thread's 32 values span 1024 / p blocks, the butterflies stay inside each); exchange
// in plain order; phase C, for one position per thread the M-point sum over the blocks in ascending order (rows with the
// same signs up to a block share its partial sum: 332 adds for M = 20), Eq. 1, and an exchange inside quads of lanes that
// turns the codes of four rows at one position into those of one row at four positions, a dword to store.  A row need not
// fill its last super-block: the missing part is never written, and what phase B reads of it stays in register groups of
// its own that are not used.
// Bound by vector issue where many rows are in flight: two waves of a SIMD issue side by side (one vector instruction in 2.1 cycles
// instead of 4.2) only while both are at plain ones, and a sub-dword, lane-move, packed or mixed-precision instruction of either
// also sets them one behind the other for long after.  MANY, for more than two rows per unit, therefore converts the inputs
// plainly and gathers the codes' bytes with permutes (v_cvt_f32_f16, v_perm_b32: more instructions than v_fma_mix_f32 and sub-dword
// adds, which calls of few rows keep for their shorter chain), and the first exchange turns its 16-byte pieces instead of padding
// rows, so that a row takes 20 KB of LDS and a unit holds 8 of order 5120 instead of 7.  16384 rows of 5120 values 70.0 -> 64.3 us
// (3.9 TB/s), 3000 17.1 -> 15.6, 1600 11.3 -> 9.8; of 2560 42.7 -> 37.8, of 1536 22.3 -> 21.5, of 3072 38.2 -> 36.7.  By the counters a
// SIMD takes 3.0 cycles per vector instruction at 35.8 a value, 4.1 at 32.3 before.  One position per thread in phase C instead of
// two: 69.9 -> 66.4 before that.  There the lane moves of all words stand in one burst at raised priority, and phases A and B, in which
// a part of the waves works and the others wait, run at raised priority too: 8000 rows of 10240 values 67.1 -> 63.3 us, 600 8.85 ->
// 8.23, 800 of 6144 6.27 -> 5.86, 1500 of 2560 6.14 -> 5.82; 16384 of 5120 level (not with blocks of 1024 values, 4000 rows of
// 12288 42.6 -> 43.1).
// Plain stores: non-temporal ones take up to 13 % off the transform alone and put more on the reader of the codes (with an int8
// product of 2560 columns behind, plain / non-temporal: 2867 rows of 5120 79.3 / 83.5 us, 13653 of 1536 95 / 105, 8192 of 2560
// 97 / 108, 3413 of 6144 91 / 96; 1000 to 1700 rows of 5120 46.8 / 45.6, 63.2 / 61.6).
// Not faster: a wave to a row, its butterflies between lanes as v_fmac_f32_dpp and lane swizzles without LDS or barriers (77 to 82 us
// for 16384 rows of 5120); s_nop around the instructions named above (69 against 69); a loop over rows with the next one's loads in flight (74.4); the sums of 4 to 16 of the
// rows as v_mfma_f32_4x4x1_16b_f32, bit for bit the same (70 to 79 against 65).
// POS = 2 is phase C with two positions per thread and 2-byte stores, a whole line of a row from every wave (launch_mixed says
// where it is the better one).
// Turned or padded pieces in the first exchange: turned where many rows are in flight, for LDS's sake, and in short calls of orders
// 12 * 128 and 20 * 128 (256 rows of 1536 values, padded / turned 3.16 / 3.03 us, of 2560 3.75 / 3.57; longer blocks are level to
// 4 % slower, 64 rows of 12288 4.26 / 4.42, but for 512 rows of 10240, 7.95 / 7.47).
template <int LOGP, bool MANY>
constexpr bool mixed_turned() { return MANY || LOGP == 7; }

template <int M, int LOGP, int POS, int ROWS, bool MANY>
__global__ void hadamard_quantize_mixed_fast_kernel(const uint16_t *y, int8_t *out, float inv_s, int64_t rows)
{
    // the ROWS rows of a workgroup are one line of N values to phases A and B, which stay inside blocks of P
    constexpr int P = 1 << LOGP, N = ROWS * M * P, T = N / 32, NSB = (N + 1023) / 1024;
    constexpr bool kTurned = mixed_turned<LOGP, MANY>(), kBursts = MANY && LOGP < 10;
    extern __shared__ float lds[];  // NSB * (kTurned ? 1024 : 1152) floats
    if (kBursts) __builtin_amdgcn_s_setprio(1);
    int t = threadIdx.x;
    size_t row = (size_t)blockIdx.x * N;
    const int here = ROWS == 1 ? 1 : (int)min((int64_t)ROWS, rows - (int64_t)blockIdx.x * ROWS);  // the last workgroup may have fewer
    if (t < (ROWS == 1 ? T : here * (M * P / 32))) {
        float v[32];
        const u32x4 *src = reinterpret_cast<const u32x4 *>(y + row + 32 * t);
        u32x4 nx[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) nx[q] = src[q];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t w = nx[q][i];
                if (!MANY) {
                    asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(v[8 * q + 2 * i]) : "v"(w));
                    asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]"
                        : "=v"(v[8 * q + 2 * i + 1]) : "v"(w));
                    continue;
                }
                uint32_t high;
                asm("v_lshrrev_b32 %0, 16, %1" : "=v"(high) : "v"(w));
                const float a = (float)__builtin_bit_cast(_Float16, (uint16_t)w);
                const float b = (float)__builtin_bit_cast(_Float16, (uint16_t)high);
                v[8 * q + 2 * i] = a + b;
                v[8 * q + 2 * i + 1] = a - b;
            }
        butterflies<5, 2>(v);
        if (kTurned) {  // value k of the thread lies in row k, whose 16-byte pieces change places with the low bits of k
            float *pa = lds + 1024 * (t >> 5) + (t & 3);
            const int piece = t >> 2 & 7;
#pragma unroll
            for (int k7 = 0; k7 < 8; ++k7) {
                float *row_k = pa + 4 * (piece ^ k7);
#pragma unroll
                for (int k = k7; k < 32; k += 8) row_k[32 * k] = v[k];
            }
        } else {
            float *pa = lds + (t & 31) + 1152 * (t >> 5);
#pragma unroll
            for (int k = 0; k < 32; ++k) pa[36 * k] = v[k];
        }
    }
    __syncthreads();
    const int t_lo = t & 31, t_hi = t >> 5;
    float v[32];
    if (t_hi < NSB) {
        // phase B: values i = t_lo + 32 e + 1024 t_hi, e = 0..31; e's low LOGP - 5 bits are the strides 32..p/2
        const f32x4 *pb = reinterpret_cast<const f32x4 *>(lds + (kTurned ? 32 : 36) * t_lo + (kTurned ? 1024 : 1152) * t_hi);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const f32x4 w = pb[kTurned ? q ^ (t_lo & 7) : q];
            v[4 * q] = w[0]; v[4 * q + 1] = w[1]; v[4 * q + 2] = w[2]; v[4 * q + 3] = w[3];
        }
        butterflies<LOGP - 5>(v);
    }
    __syncthreads();  // all reads of the transposed layout are done before the plain one overwrites it
    if (t_hi < NSB) {
        float *pb = lds + t_lo + 1024 * t_hi;
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if (1024 * t_hi + 32 * e < N) pb[32 * e] = v[e];  // uniform per wave half: whole groups of 32 lanes
    }
    __syncthreads();
    if (kBursts) __builtin_amdgcn_s_setprio(0);
    const float *line = lds;
    if (ROWS > 1) {
        const int r = t >> (LOGP + 1 - POS);
        if (r >= here) return;
        t &= P / POS - 1;
        line += r * (M * P);
        row += (size_t)r * (M * P);
    }
    if constexpr (POS == 2) {
        // phase C: positions 2 t and 2 t + 1 of every block
        float t0[M], t1[M];
#pragma unroll
        for (int b = 0; b < M; ++b) {
            t0[b] = line[b * P + 2 * t];
            t1[b] = line[b * P + 2 * t + 1];
        }
#pragma unroll
        for (int a = 0; a < M; ++a) {
            float a0 = t0[0] * paley_sign<M>(a, 0), a1 = t1[0] * paley_sign<M>(a, 0);
#pragma unroll
            for (int b = 1; b < M; ++b) {
                a0 = a0 + t0[b] * paley_sign<M>(a, b);
                a1 = a1 + t1[b] * paley_sign<M>(a, b);
            }
            const float sc[4] = {a0 * inv_s, a1 * inv_s, 0.0f, 0.0f};
            *reinterpret_cast<uint16_t *>(out + row + (size_t)a * P + 2 * t) = (uint16_t)codes_gathered<2>(sc);
        }
    } else {
        // phase C: position t of every block, four rows of the M-point sums at a time
        float x[M];
#pragma unroll
        for (int b = 0; b < M; ++b) x[b] = line[b * P + t];
        int8_t *dst = out + row + (size_t)(t & 3) * P + (t & ~3);
        const uint32_t sel1 = t & 1 ? 0x03070105u : 0x06020400u, sel2 = t & 2 ? 0x03020706u : 0x05040100u;
        uint32_t w[M / 4];
#pragma unroll
        for (int a = 0; a < M; a += 4) {
            float sc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float acc = x[0] * paley_sign<M>(a + i, 0);
#pragma unroll
                for (int b = 1; b < M; ++b) acc = acc + x[b] * paley_sign<M>(a + i, b);
                sc[i] = acc * inv_s;
            }
            w[a / 4] = MANY ? codes_gathered<4>(sc) : codes_packed<4>(sc);
            if (!kBursts) {
                // a lane's dword holds the codes of rows a .. a + 3; after the exchange inside the quad, of four positions of row
                // a + t % 4
                const uint32_t w1 = __builtin_amdgcn_perm(__builtin_amdgcn_update_dpp(0u, w[a / 4], 0xB1, 0xf, 0xf, true), w[a / 4], sel1);
                const uint32_t w2 = __builtin_amdgcn_perm(__builtin_amdgcn_update_dpp(0u, w1, 0x4E, 0xf, 0xf, true), w1, sel2);
                *reinterpret_cast<u32_u *>(dst + (size_t)a * P) = w2;
            }
        }
        if constexpr (kBursts) {  // the same exchange of all rows
            uint32_t other[M / 4];
            swap_lanes<0>(w, other);
#pragma unroll
            for (int k = 0; k < M / 4; ++k) w[k] = __builtin_amdgcn_perm(other[k], w[k], sel1);
            swap_lanes<1>(w, other);
#pragma unroll
            for (int k = 0; k < M / 4; ++k)
                *reinterpret_cast<u32_u *>(dst + (size_t)(4 * k) * P) = __builtin_amdgcn_perm(other[k], w[k], sel2);
            __builtin_amdgcn_s_setprio(0);
        }
    }
}

template <int M, int LOGP, int POS, int ROWS, bool MANY>
hipError_t launch_mixed_form(const uint16_t *y, int64_t rows, float inv_s, int8_t *out, hipStream_t stream)
{
    constexpr int P = 1 << LOGP, N = ROWS * M * P, NSB = (N + 1023) / 1024;
    constexpr int threads = ROWS * P / POS;
    static_assert(POS == 1 || MANY, "two positions only on large calls");
    static_assert(threads >= N / 32 && threads >= 32 * NSB, "every phase has its threads");
    constexpr int lds = NSB * (mixed_turned<LOGP, MANY>() ? 1024 : 1152) * (int)sizeof(float);
    static_assert(threads <= 1024 && lds <= 160 * 1024, "launch shape");
    if (lds > 48 * 1024) {
        const hipError_t e = allow_full_lds<hadamard_quantize_mixed_fast_kernel<M, LOGP, POS, ROWS, MANY>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((hadamard_quantize_mixed_fast_kernel<M, LOGP, POS, ROWS, MANY>), dim3((unsigned)((rows + ROWS - 1) / ROWS)),
                       dim3(threads), lds, stream, y, out, inv_s, rows);
    return hipGetLastError();
}

template <int M, int LOGP>
hipError_t launch_mixed(const uint16_t *y, int64_t rows, float inv_s, int8_t *out, hipStream_t stream)
{
    // More than 16 rows per unit: several to a workgroup where the waves of one would be left partly idle in phases A and B (48, 80 and 96
    // threads' work).  One row / several (us): order 2560, 2600 rows 8.70 / 8.96, 5000 13.9 / 13.2, 16384 38.4 / 34.8; 1536: 5000 8.17 /
    // 8.22, 10000 13.2 / 12.8, 16384 19.1 / 18.4; 3072: 3000 8.99 / 9.19, 6000 15.2 / 14.8, 16384 38.2 / 37.1.  Order 5120 has 160
    // threads' work for 3 waves and loses more by the longer barriers than it gains (16384 rows 66.4 / 67.3).
    const bool many_more = rows > 16 * (int64_t)compute_units();
    // Two positions on large calls of orders 12 * 128 .. 12 * 512 (order 12 * 1024 gains from one position at every size, 20 * 2^k has
    // no threads to spare with two).  12 * 256 and 12 * 512 whose codes outgrow the caches of the dies: half lines cost more than
    // the waves gain (order 6144, one / two positions: 498 rows 3.97 / 4.12 us, 822 5.94 / 5.92, 909 6.49 / 6.16, 14336 54.9 / 51.0;
    // order 3072: 1488 rows 5.65 / 5.84, 1645 6.01 / 5.97, 1818 6.48 / 6.31, 28672 57.0 / 53.3).  12 * 128 while the rows are more
    // than 9 of the 16 workgroups that a unit holds with one position (2204 rows 4.41 / 4.66, 2436 4.96 / 4.85, 3637 6.53 / 6.09,
    // 4020 6.88 / 6.56, 4443 7.59 / 7.71).
    if constexpr (M == 12 && (LOGP == 8 || LOGP == 9))
        if (rows * M * (1 << LOGP) > 5LL << 20) {
            if (LOGP == 8 && many_more) return launch_mixed_form<M, LOGP, 2, LOGP == 8 ? 2 : 1, true>(y, rows, inv_s, out, stream);
            return launch_mixed_form<M, LOGP, 2, 1, true>(y, rows, inv_s, out, stream);
        }
    if constexpr (M == 12 && LOGP == 7)
        if (rows > 9 * compute_units() && rows <= 16 * compute_units())
            return launch_mixed_form<M, LOGP, 2, 1, true>(y, rows, inv_s, out, stream);
    // More than two rows per compute unit: enough waves for a SIMD's vector instructions to count.  (Order 5120, the short forms / these:
    // 512 rows 5.04 / 5.10 us, 600 6.30 / 5.87, 1600 11.3 / 9.8, 16384 70.0 / 64.3; 12288: 256 rows 5.41 / 5.53, 800 12.57 / 12.35.
    // One line for all orders: on inputs that lie in the caches, calls just above it lose up to 1.7 %, 520 rows of 3072 3.58 / 3.62.)
    if (LOGP == 7 && many_more) return launch_mixed_form<M, LOGP, 1, LOGP == 7 ? 4 : 1, true>(y, rows, inv_s, out, stream);
    if (rows > 2 * compute_units()) return launch_mixed_form<M, LOGP, 1, 1, true>(y, rows, inv_s, out, stream);
    return launch_mixed_form<M, LOGP, 1, 1, false>(y, rows, inv_s, out, stream);
}

template <int LOGN>
hipError_t launch_fast(const uint16_t *y, int64_t rows, float inv_s, int8_t *out, hipStream_t stream)
{
    constexpr int N = 1 << LOGN, RPW = rows_per_workgroup<LOGN>();
    constexpr int lds = RPW * (N / 1024) * 1152 * (int)sizeof(float);
    // twice the workgroups that fit the device at once (measured best; one round of exactly resident workgroups
    // is 10% slower), asked of the runtime once per order and device
    static std::atomic<int> resident[16];  // zero-initialised; concurrent first calls compute the same value
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 16) return hipErrorInvalidDevice;
    if (!resident[dev].load()) {
        if (lds > 48 * 1024) {
            e = allow_full_lds<hadamard_quantize_kernel<LOGN>>();
            if (e != hipSuccess) return e;
        }
        int per_cu = 0, cus = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, hadamard_quantize_kernel<LOGN>, RPW * N / 32, lds);
        if (e != hipSuccess) return e;
        cus = compute_units();
        resident[dev].store(per_cu > 0 && cus > 0 ? 2 * per_cu * cus : 2048);
    }
    const int res = resident[dev].load();
    const int64_t groups = (rows + RPW - 1) / RPW;
    const unsigned grid = (unsigned)(groups < res ? groups : res);
    hipLaunchKernelGGL(hadamard_quantize_kernel<LOGN>, dim3(grid), dim3(RPW * N / 32), lds, stream, y, out, (int)rows,
                       inv_s);
    return hipGetLastError();
}

}  // namespace

bool hadamard_order_supported(int n)
{
    if (n < 2 || n > 16384) return false;
    if ((n & (n - 1)) == 0) return true;
    for (int m : {12, 20})
        if (n % m == 0 && ((n / m) & (n / m - 1)) == 0 && n / m >= 4) return true;
    return false;
}

hipError_t launch_hadamard_quantize(const uint16_t *y, int64_t rows, int n, float s_y, int8_t *out, hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    const float inv_s = 1.0f / s_y;  // correctly rounded fp32 division on the host
    if (n & (n - 1)) {
        const int m = (n % 12 == 0 && ((n / 12) & (n / 12 - 1)) == 0) ? 12 : 20;
        if (reinterpret_cast<uintptr_t>(y) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 2 == 0) {
            switch (n) {  // the register-blocked kernel for blocks of 128 .. 1024 values
                case 12 * 128: return launch_mixed<12, 7>(y, rows, inv_s, out, stream);
                case 12 * 256: return launch_mixed<12, 8>(y, rows, inv_s, out, stream);
                case 12 * 512: return launch_mixed<12, 9>(y, rows, inv_s, out, stream);
                case 12 * 1024: return launch_mixed<12, 10>(y, rows, inv_s, out, stream);
                case 20 * 128: return launch_mixed<20, 7>(y, rows, inv_s, out, stream);
                case 20 * 256: return launch_mixed<20, 8>(y, rows, inv_s, out, stream);
                case 20 * 512: return launch_mixed<20, 9>(y, rows, inv_s, out, stream);
                default: break;
            }
        }
        const int lds = n * (int)sizeof(float);
        const int aligned = reinterpret_cast<uintptr_t>(out) % 4 == 0;
        if (m == 12) {
            if (lds > 48 * 1024) {
                const hipError_t e = allow_full_lds<hadamard_quantize_mixed_kernel<12>>();
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(hadamard_quantize_mixed_kernel<12>, dim3((unsigned)rows), dim3(256), lds, stream, y, out,
                               n / 12, inv_s, aligned);
        } else {
            if (lds > 48 * 1024) {
                const hipError_t e = allow_full_lds<hadamard_quantize_mixed_kernel<20>>();
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(hadamard_quantize_mixed_kernel<20>, dim3((unsigned)rows), dim3(256), lds, stream, y, out,
                               n / 20, inv_s, aligned);
        }
        return hipGetLastError();
    }
    const bool al = reinterpret_cast<uintptr_t>(y) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 4 == 0;
    if (al) {
        switch (n) {
            case 1024: return launch_fast<10>(y, rows, inv_s, out, stream);
            case 2048: return launch_fast<11>(y, rows, inv_s, out, stream);
            case 4096: return launch_fast<12>(y, rows, inv_s, out, stream);
            case 8192: return launch_fast<13>(y, rows, inv_s, out, stream);
            case 16384: return launch_fast<14>(y, rows, inv_s, out, stream);
            default: break;
        }
    }
    const int lds = n * (int)sizeof(float);
    if (lds > 48 * 1024) {
        const hipError_t e = allow_full_lds<hadamard_quantize_small_kernel>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(hadamard_quantize_small_kernel, dim3((unsigned)rows), dim3(256), lds, stream, y, out, n, inv_s);
    return hipGetLastError();
}

}  // namespace quamba
