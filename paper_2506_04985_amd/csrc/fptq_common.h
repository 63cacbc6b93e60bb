// Shared declarations of the fptq HIP library (gfx950 only): packed layout arithmetic, error
// reporting, and the launcher prototypes that tie the translation units together.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "fptq.h"

namespace fptq {

// Packed INT4 layout: K is cut into tiles of KT values; each (tile, row) pair owns one
// 64-byte segment, tiles outermost.  Within a segment value k sits in byte (k % KT) / 2,
// low nibble first.
constexpr int KT = 128;          // values per K tile
constexpr int SEG = KT / 2;      // bytes per (row, tile) segment

__host__ __device__ inline int64_t k_tiles(int64_t K) { return (K + KT - 1) / KT; }
__host__ __device__ inline int64_t packed_bytes(int64_t rows, int64_t K) { return k_tiles(K) * rows * SEG; }

// error text of the calling thread (set by the API layer)
void set_error(const char *fmt, ...);

// kernel launchers (each returns a hipError_t from hipGetLastError after the launch)
hipError_t launch_pack_weights(const int8_t *w, int64_t N, int64_t K, uint8_t *out, hipStream_t s);
hipError_t launch_unpack(const uint8_t *packed, int64_t rows, int64_t K, int8_t *out, hipStream_t s);
hipError_t launch_quantize_act(const uint16_t *x, int64_t M, int64_t K, int mode, float eps, const float *row_in,
                               float inv_s_a, int zero_point, uint8_t *out, float *row_out, hipStream_t s);
hipError_t launch_residual_norm_quantize(const uint16_t *xr, const uint16_t *yb, int64_t M, int64_t K, const float *s_prev,
                                         float eps, float inv_s_a, uint16_t *x_next, float *s_next, uint8_t *out, hipStream_t s);
hipError_t launch_weight_row_sums(const int8_t *w, int64_t N, int64_t K, int32_t *sums, hipStream_t s);
hipError_t launch_quantize_act_dynamic(const uint16_t *x, int64_t M, int64_t K, uint8_t *out, float *s_out, hipStream_t s);
hipError_t launch_quantize_act_hadamard(const uint16_t *x, int64_t M, int64_t K, int hadamard_block, int mode, float eps,
                                        const float *row_in, float inv_s_a, uint8_t *out, float *row_out, hipStream_t s);
hipError_t launch_linear_ref(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                             const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                             hipStream_t s);
hipError_t launch_linear_mfma(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                              const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                              hipStream_t s);
hipError_t launch_linear_mfma_ws(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                                 const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                                 int32_t *ws, int64_t ws_bytes, hipStream_t s);
int64_t linear_workspace_bytes(int64_t M, int64_t N, int64_t K);
hipError_t launch_linear_prefill(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a, const float *s_w,
                                 const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc, uint8_t *scratch, int tile_tokens,
                                 hipStream_t s);
int64_t prefill_scratch_bytes(int64_t M, int64_t K);
int64_t prefill_workgroups(int64_t M, int64_t N, int tile_tokens);
int prefill_tile(int64_t M, int64_t N, int64_t K);      // tokens per tile (256, 192 or 128), 0 where another kernel is faster
hipError_t launch_linear_decode(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                                const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                                hipStream_t s);

void set_gemm_tile(int tile);
void set_gemm_map(int mode);
void set_linear_prefill(int mode);
int forced_gemm_tile();
bool set_decode_shape(int code);

// What a linear call would launch: kernel (template instance or name), workgroups, threads per workgroup.
struct LinearPlan {
    char kernel[96];
    int64_t workgroups;
    int threads;
};
void linear_mfma_plan(int64_t M, int64_t N, int64_t K, bool with_workspace, LinearPlan *plan);

// Per-device state, set up once per device (by fptq_init or by the first call that needs it; thread-safe):
// the number of compute units, which the launchers size their grids and pick their tile shapes by, and the
// device address of the library's built-in scratch area (fptq_w4a4_linear_noalloc).
constexpr int MAX_DEVICES = 64;
constexpr int DEFAULT_CUS = 256;                 // MI355X; used by the host-only size queries when no device answers
struct DeviceInfo {
    int device;
    int cus;
    int32_t *scratch;
    int64_t scratch_bytes;
};
hipError_t device_info(const DeviceInfo **out);  // state of the current device
int device_cus_or_default();                     // compute units of the current device, DEFAULT_CUS without one
// what each translation unit contributes to that set-up (called with the device current, under the set-up lock)
hipError_t gemm_device_init(DeviceInfo *info);
hipError_t prefill_device_init();

// ---- what several kernel sources share

typedef int v4i __attribute__((ext_vector_type(4)));

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// s_waitcnt immediates for gfx9: vmcnt in bits [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int WAIT_LGKM0 = 15 | (3 << 14) | (7 << 4) | (0 << 8);

// raw buffer descriptor, dword 3: 32-bit data format, no swizzle (gfx9 family encoding); reads past num_records return zero
constexpr int RSRC_FLAGS = 0x00020000;

// two fp32 -> packed bf16 pair (round to nearest even, hardware conversion)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16(float lo, float hi)
{
    float2_t f = {lo, hi};
    bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
    return __builtin_bit_cast(uint32_t, b);
}

// fp32 -> bf16 bit pattern, round to nearest even (NaN stays a quiet NaN)
__device__ inline uint16_t bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Chunks of eight bf16 values of a row, from k0 on every `step` values, zeros past the row's end: 16-byte loads at any alignment (the hardware
// takes it).  A chunk that would reach past the end is loaded from eight values before it and shifted, so that no lane loads by element and
// no branch keeps a chunk's load behind another's: rows of few values are one latency long.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
template <int CH>
__device__ inline void load_row_chunks(v4u (&v)[CH], const uint16_t *row, int k0, int step, int K)
{
    const int last = K - 8;
    if (last < 0) {
        uint32_t e[8] = {};
#pragma unroll
        for (int i = 0; i < 7; ++i) e[i] = row[min(i, K - 1)];
#pragma unroll
        for (int i = 0; i < 7; ++i) e[i] = k0 == 0 && i < K ? e[i] : 0u;
#pragma unroll
        for (int i = 0; i < CH; ++i) v[i] = v4u{0, 0, 0, 0};
        v[0] = v4u{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6]};
        return;
    }
#pragma unroll
    for (int i = 0; i < CH; ++i) __builtin_memcpy(&v[i], row + min(k0 + i * step, last), 16);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int s = k0 + i * step - last;          // values that lie in front of the chunk
        if (s > 0) {
            v4u a = v[i];
            if (s & 4) a = v4u{a.z, a.w, 0, 0};
            if (s & 2) a = v4u{a.y, a.z, a.w, 0};
            if (s & 1) a = v4u{a.x >> 16 | a.y << 16, a.y >> 16 | a.z << 16, a.z >> 16 | a.w << 16, a.w >> 16};
            v[i] = s < 8 ? a : v4u{0, 0, 0, 0};
        }
    }
}

// HIP refuses a launch of 2^32 threads or more: waves of a launch of workgroups of 256 threads.  Kernels that spread a row over more waves
// than another one that serves it leave calls beyond that to the other.
constexpr int64_t MAX_WAVES = ((int64_t)1 << 26) - 4;

// Many short rows: a wave takes a row, where a workgroup per row (which spreads a row over four waves) has most of its threads idle or more
// waves than the device runs at once.  Aligned rows: crossover at 4096 values about 1000 rows with RMS scale (4096 x 4096 from HBM 11.0 us with a wave,
// 10.8 with a workgroup, from the last-level cache 8.8 and 9.5); the residual step and the dynamic scale, which have more to do per value, take a workgroup for
// some rows above 3072 values, by lines of their own (4096 x 4096, wave / workgroup, from HBM and from the cache: 21.2 / 20.0, 17.0 / 17.3 and 11.0 / 10.4, 8.9 / 8.8; 4096 x
// 3072 18.3 / 17.2, 13.7 / 14.6).  Ragged ones (workgroup / wave, RMS scale): 800 x 63
// 3.3 / 2.3 us, 2048 x 333 4.6 / 2.7, 65536 x 63 82 / 23, 4000 x 3601 11.8 / 10.0; residual step 8192 x 333 19 / 6.7; but dynamic scale 1100 x 3601
// 5.1 / 6.2, given scale 2048 x 1801 3.6 / 4.1.
inline bool wave_per_row(bool vec, int64_t M, int64_t K, int64_t longest_aligned = 4096)
{
    return K <= (vec ? longest_aligned : 4096) && M > (vec || K <= 1024 ? 768 : 3072);
}

// Its instances: CASE(chunks a lane, ragged).  Ragged rows in finer steps, because a chunk that lies past the row's end is loaded and computed
// all the same (800 x 777, residual step: 5.1 us with four chunks, 3.8 with two).
#define WAVE_PER_ROW_RAGGED(K, CASE)                      \
    do {                                                  \
        if ((K) <= 512) CASE(1, true);                    \
        else if ((K) <= 1024) CASE(2, true);              \
        else if ((K) <= 2048) CASE(4, true);              \
        else if ((K) <= 3072) CASE(6, true);              \
        else CASE(8, true);                               \
    } while (0)
#define WAVE_PER_ROW(vec, K, CASE)                        \
    do {                                                  \
        if (!(vec)) WAVE_PER_ROW_RAGGED(K, CASE);         \
        else if ((K) <= 2048) CASE(4, false);             \
        else CASE(8, false);                              \
    } while (0)

// a / n and a % n with m = reciprocal(n), in a few scalar instructions: the estimate is the quotient or one less (the division that the compiler makes of
// a run-time divisor is a chain of twenty, 0.1 us at the start of every wave)
inline uint32_t reciprocal(uint32_t n) { return n == 1 ? 0xffffffffu : (uint32_t)(((uint64_t)1 << 32) / n); }
__device__ inline void divide(uint32_t a, uint32_t n, uint32_t m, uint32_t &quotient, uint32_t &remainder)
{
    const uint32_t q = __umulhi(a, m), r = a - q * n;
    quotient = r >= n ? q + 1 : q, remainder = r >= n ? r - n : r;
}

// what of a word of eight codes from k0 on lies inside the row: K padding stays zero
__device__ inline uint32_t codes_inside(uint32_t word, int k0, int K)
{
    return k0 + 8 <= K ? word : k0 < K ? word & ((1u << (4 * (K - k0))) - 1u) : 0u;
}

// ss + v * v in fp64 for an fp32 v: the square of a value with at most 24 significant bits is exact in fp64, so the
// fused form rounds once, exactly like the separate multiply and add of the definition.
__device__ inline double add_square(double ss, float v)
{
    const double a = (double)v;
    return __builtin_fma(a, a, ss);
}

// Wave reductions, every lane with the result: partners 32, 16, 8, 4, 2, 1 lanes away, in the order of a loop over __shfl_xor (sums of
// doubles round the same way), but without its round trips through LDS, six for a sum and twice as many instructions for doubles: with
// few rows a quantizer's time is one such chain of latencies.
template <int OFF>
__device__ inline uint32_t other_lane(uint32_t v)        // of lane ^ OFF, OFF < 16
{
    if (OFF == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);              // row_ror:8
    if (OFF == 4) {                                                                                             // row_shl:4, row_shr:4
        const int up = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x104, 0xF, 0x5, false);
        return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)v, 0x114, 0xF, 0xA, false);
    }
    if (OFF == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);               // quad_perm [2,3,0,1]
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);                             // quad_perm [1,0,3,2]
}

template <bool ALL = true>                               // else: every lane with the sum of those whose bit 4 is the same
__device__ inline double wave_sum(double v)
{
    auto join = [](uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo); };
    auto lo = [](double d) { return (uint32_t)__builtin_bit_cast(uint64_t, d); };
    auto hi = [](double d) { return (uint32_t)(__builtin_bit_cast(uint64_t, d) >> 32); };
    // a swap of a register with itself leaves the values of one side of each pair in the first result, of the other in the second
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo(v), lo(v), false, false), h32 = __builtin_amdgcn_permlane32_swap(hi(v), hi(v), false, false);
    v = join(l32[0], h32[0]) + join(l32[1], h32[1]);
    if (ALL) {
        const auto l16 = __builtin_amdgcn_permlane16_swap(lo(v), lo(v), false, false), h16 = __builtin_amdgcn_permlane16_swap(hi(v), hi(v), false, false);
        v = join(l16[0], h16[0]) + join(l16[1], h16[1]);
    }
    v += join(other_lane<8>(lo(v)), other_lane<8>(hi(v)));
    v += join(other_lane<4>(lo(v)), other_lane<4>(hi(v)));
    v += join(other_lane<2>(lo(v)), other_lane<2>(hi(v)));
    v += join(other_lane<1>(lo(v)), other_lane<1>(hi(v)));
    return v;
}

__device__ inline uint32_t wave_max(uint32_t v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max(b[0], b[1]);
    v = max(v, other_lane<8>(v));
    v = max(v, other_lane<4>(v));
    v = max(v, other_lane<2>(v));
    return max(v, other_lane<1>(v));
}

// Core of every activation quantizer: the code q + 8 in [0, 15] of q = clamp(rne(x * c) + z, -8, 7), NaN -> z,
// with zoff = z + 8.  v_cvt_i32_f32 saturates and turns NaN into 0, the add saturates too, so infinities and
// huge products end at the clamp like everything else: the same integers as rounding, adding and clamping in
// float.  XOR with 8 turns the code into the two's complement nibble (eight at a time: CODE_TO_NIBBLES).
__device__ inline uint32_t quant_code(float x, float c, int zoff)
{
    const float r = __builtin_rintf(x * c);
    int i, j;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(i) : "v"(r));
    asm("v_add_i32 %0, %1, %2 clamp" : "=v"(j) : "v"(i), "v"(zoff));
    return (uint32_t)min(max(j, 0), 15);
}
constexpr uint32_t CODE_TO_NIBBLES = 0x88888888u;

// The same codes on the symmetric grid in 3.25 instructions a value instead of 6, for products x * c that are no NaN: clamped between the grid's
// ends first (integers, so the order does not matter), then rounded by adding 1.5 * 2^23, whose sum holds the code in its low bits, written to a byte of a
// register at once; the even values' bytes and the odd ones' make the word of nibbles, value e in nibble e.  Two writes to one register need a
// wait state between them, and so does its first reader.
__device__ inline uint32_t quantize_tame(const float *x, float c)
{
    float t[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = __builtin_amdgcn_fmed3f(x[e] * c, -8.0f, 7.0f);
    uint32_t even, odd;
    asm("v_add_f32_sdwa %0, %2, %10 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %1, %3, %10 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %0, %4, %10 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %1, %5, %10 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %0, %6, %10 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %1, %7, %10 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %0, %8, %10 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "v_add_f32_sdwa %1, %9, %10 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "s_nop 0"
        : "=&v"(even), "=&v"(odd)
        : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "v"(12582912.0f));
    return (even & 0x0F0F0F0Fu) | (odd << 4 & 0xF0F0F0F0u);
}

// What shows that no product is a NaN: a sum of squares of the inputs (two to an instruction) below TAME bounds them by 2^62, so the sums of any 4096 of
// them are finite, and so is a multiplier below it.
constexpr float TAME = 0x1p123f;
__device__ inline float add_squares(float sum, uint32_t pair)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair), __builtin_bit_cast(bf16x2_t, pair), sum, false);
}

// Zero-point correction of an accumulator: sum_k (v - z) w = acc - z * sum_k w (wsum == NULL: symmetric grid).
__device__ inline int32_t remove_zero_point(int32_t acc, int zp, const int32_t *wsum, int64_t o)
{
    return wsum ? acc - zp * wsum[o] : acc;
}

// How a matrix kernel's results reach memory.  Rows of whole 64-byte pieces are streamed (six-bit kernel, 8192 x 57344 x 8192: zeros 1090 us, cached
// 1365; dense 1632 and 1658; INT8 kernel, 1000 x 5120 x 4096 22.9 and 23.7, 300 x 20000 x 1000 11.8 and 12.7).  Other widths leave two
// parts of a piece to two waves, which meet in L2 when cached; streamed, each goes to memory by itself: 3000 x 11000 x 2048 76 us, cached
// 66, 4096 x 4104 x 4096 70 and 65, 1000 x 9000 x 3000 36 and 34, on the INT8 kernel 333 x 32008 x 2504 30.2 and 29.7.  An output that the
// 256 MB last-level cache cannot hold is streamed all the same if its rows are multiples of 16 bytes: cached, 8192 x 28680 x 1024 took 271 us instead of
// 255, 8192 x 16392 x 2048 213 instead of 203.  Other rows are cached at any size: streamed, 8192 x 32003 x 1024 takes 319 us instead of 251, 4096 x
// 32003 x 4096 300 instead of 283, 3000 x 11001 x 2048 80 instead of 66, 2048 x 128257 x 2048 391 instead of 389 (INT8 kernel 291 and 276, 382 and 382, 71
// and 65, 435 and 444).  64 bytes are half a line: on the six-bit kernel rows of an odd number of them lose up to 3 % streamed (3000 x 11040 x 2048 56.7 us,
// cached 55.0, 4096 x 4128 x 4096 55.0 and 54.1) and gain 5 % where the output is large (4096 x 28704 x 1024 112 and 118, 8192 x 14368 x 1024 116 and 121).
enum { ANY_ALIGNMENT, CACHED, STREAMED };          // ANY_ALIGNMENT: serves every N, chosen for N % 8 != 0
inline int store_kind(int64_t M, int64_t N)
{
    return N % 8 != 0 ? ANY_ALIGNMENT : N % 32 != 0 && M * N * 2 <= (int64_t)256 << 20 ? CACHED : STREAMED;
}
constexpr int NON_TEMPORAL = 2;                    // cache policy of a buffer access

// Stores a wave's row segments of 32 tokens from mt0 on: pass p takes ROWS_PER_PASS rows, this lane channels nn .. nn + 7 of row
// p * ROWS_PER_PASS + row.  y_off: the lane's byte offset in the first pass, or one past every descriptor's end if its segment is not whole or not
// there; rows past M fail the descriptor's check.  edge: the row's end falls into this wave's channels.
template <int STORE, int PASSES, int ROWS_PER_PASS>
__device__ inline void store_rows(const uint4 (&v)[PASSES], uint16_t *y, uint32_t y_off, int mt0, int row, int nn, bool live, int M, int N, bool edge)
{
    const uint32_t row_stride = (uint32_t)N * 2, bytes = (uint32_t)max(0, min(32, M - mt0)) * row_stride;      // 2^30 at most: N <= 2^24
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(y + (int64_t)mt0 * N, 0, __builtin_amdgcn_readfirstlane((int)bytes), RSRC_FLAGS);
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        __builtin_amdgcn_raw_buffer_store_b128(v4i{(int)v[p].x, (int)v[p].y, (int)v[p].z, (int)v[p].w}, yr, y_off + p * ROWS_PER_PASS * row_stride, 0,
                                               STORE == STREAMED ? NON_TEMPORAL : 0);
    if (STORE == ANY_ALIGNMENT && edge) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (live && nn + 8 > N && mt0 + p * ROWS_PER_PASS + row < M) {
                const uint32_t w[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
                uint16_t *const dst = y + (int64_t)(mt0 + p * ROWS_PER_PASS + row) * N + nn;
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (nn + e < N) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
            }
    }
}

// The dequantizing epilogue of the layer for one output: fp32 throughout, no fused operations.
__device__ inline uint16_t dequant_bf16(int32_t acc, float cw, const float *d, int64_t t)
{
    float yf = (float)acc * cw;
    if (d) yf = yf * d[t];
    return bf16_rne(yf);
}

}  // namespace fptq
