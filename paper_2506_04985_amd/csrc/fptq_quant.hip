// Activation path of the quantized linear layer: per-token scale (Sec. 3.1.3 Step 1), static
// per-tensor INT4 quantization (App. B) and nibble packing (App. J) in one pass over X.
//
// The row is read once from HBM and kept in registers while the sum of squares is reduced, then
// quantized from the registers.  Bandwidth-bound: 2 bytes read and half a byte written per
// element.  Short rows in large numbers are handled by one wave each (no LDS, no barrier, the scale is
// computed once per row, and many rows are in flight per CU); longer rows, or few, by one workgroup each.  Where the scale is given there
// is nothing to reduce and a wave takes a piece of a row.
#include <type_traits>

#include "fptq_common.h"

namespace fptq {

constexpr int QT = 256;        // threads per row
constexpr int QCHUNK = 8;      // bf16 values per 16-byte load

__device__ inline float bf16_to_f32(uint32_t bits) { return __uint_as_float(bits << 16); }

// Eight quantized values of one 16-byte chunk of bf16 as a packed word (value e in nibble e).
__device__ inline uint32_t quant_chunk(const uint32_t (&w)[4], float c, int zoff)
{
    uint32_t word = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        word |= quant_code(bf16_to_f32(w[j] & 0xffffu), c, zoff) << (8 * j);
        word |= quant_code(bf16_to_f32(w[j] >> 16), c, zoff) << (8 * j + 4);
    }
    return word ^ CODE_TO_NIBBLES;
}

__device__ inline double block_sum(double v, double *lds)
{
    v = wave_sum(v);
    int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) lds[wave] = v;
    __syncthreads();
    double tot = lds[0];
#pragma unroll
    for (int w = 1; w < QT / 64; ++w) tot += lds[w];
    return tot;
}

__device__ inline void store_word(uint8_t *out, int64_t M, int64_t t, int64_t k0, uint32_t word)
{
    *reinterpret_cast<uint32_t *>(out + ((k0 / KT) * M + t) * SEG + (k0 % KT) / 2) = word;
}

typedef v4u q_v4u;
constexpr int Q_STREAM = 2;      // buffer-load cache policy: non-temporal

// One workgroup per row.  CH > 0: K % 8 == 0, 16-byte aligned rows of at most 2048 * CH values, kept in
// registers (CH 16-byte chunks per thread) between the reduction and the quantizer and read through a row-sized
// buffer descriptor, so chunks past the end read as zero and nothing branches but the store of a chunk past
// the padded width.  RAGGED: the same for any K and alignment, each chunk loaded where it lies (RMS scale: 279 x 11849 21.8 us in two passes by
// element, now 6.1, 2048 x 4366 19.1 and 8.7).  CH == 0: rows too long for the registers, two passes over the row.
//
// Arguments: the first 14 words of a kernel's arguments come with the dispatch, and a wait for one beyond them is a memory latency at the start of
// every wave; so the width is one word where the row fits the registers, and zoff has the input's streaming in its second byte.  With that
// flag as the 17th word / without any argument preloaded / now, measured when this kernel still served aligned rows of a given scale: 4096 x 4096 9.5, 9.8,
// 9.15 us, 256 x 8192 3.3, 3.3, 3.1, 32 x 4096 2.34, 2.32, 2.28.
template <int CH> using width_t = std::conditional_t<(CH > 0), int, int64_t>;
constexpr int STREAM_IN = 256;

template <int MODE, int CH, bool RAGGED>
__global__ __launch_bounds__(QT) void quantize_act_kernel(const uint16_t *__restrict__ x, uint8_t *__restrict__ out, float *__restrict__ row_out,
                                                          const float *__restrict__ row_in, int64_t M, width_t<CH> K, float inv_s_a, int zoff_stream,
                                                          float eps)
{
    const int zoff = zoff_stream & 255, stream_in = zoff_stream & STREAM_IN;
    __shared__ double red[QT / 64];
    const int64_t t = blockIdx.x;
    const uint16_t *row = x + t * K;
    const int64_t Kpad = k_tiles(K) * KT;
    const int tid = threadIdx.x;

    q_v4u regs[CH > 0 ? CH : 1];
    if (RAGGED) {
        load_row_chunks(regs, row, tid * QCHUNK, QT * QCHUNK, (int)K);
    } else if (CH > 0) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, (int)K * 2, RSRC_FLAGS);
        if (stream_in) {         // an input larger than the last-level cache: streaming loads, which do not displace what is there
#pragma unroll
            for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * QT + tid) * 16, 0, Q_STREAM);
        } else {
#pragma unroll
            for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * QT + tid) * 16, 0, 0);
        }
    }

    float r = 1.0f;
    if (MODE == FPTQ_SCALE_RMS) {
        double ss = 0.0;
        if (CH > 0) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // a * a is exact in fp64 (8 significant bits squared), so the fused form rounds like multiply, then add
                    double a = (double)bf16_to_f32(w[j] & 0xffffu), b = (double)bf16_to_f32(w[j] >> 16);
                    ss = __builtin_fma(a, a, ss);
                    ss = __builtin_fma(b, b, ss);
                }
            }
        } else {
            for (int64_t k = tid; k < K; k += QT) {
                double a = (double)bf16_to_f32(row[k]);
                ss = __builtin_fma(a, a, ss);
            }
        }
        ss = block_sum(ss, red);
        r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    } else if (MODE == FPTQ_SCALE_GIVEN) {
        r = row_in[t];
    }
    const float c = (MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a;
    if (tid == 0 && row_out) row_out[t] = r;

    if (CH > 0) {
        // chunk i of thread h is values 8 (256 i + h) ..: K tile 16 i + h / 16, byte 4 (h % 16) of the row's segment
        uint8_t *orow = out + (((int64_t)(tid >> 4) * M + t) * SEG + (tid & 15) * 4);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k0 = (i * QT + tid) * QCHUNK;
            const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
            uint32_t word = quant_chunk(w, c, zoff);
            word = RAGGED ? codes_inside(word, k0, (int)K) : k0 >= (int)K ? 0u : word;      // K padding stays zero
            if (k0 < (int)Kpad) *reinterpret_cast<uint32_t *>(orow + (int64_t)(16 * i) * M * SEG) = word;
        }
    } else {
        for (int64_t k0 = (int64_t)tid * QCHUNK; k0 < Kpad; k0 += (int64_t)QT * QCHUNK) {
            uint32_t word = 0;
#pragma unroll
            for (int i = 0; i < QCHUNK; ++i) {
                int64_t k = k0 + i;
                if (k < K) word |= (quant_code(bf16_to_f32(row[k]), c, zoff) ^ 8u) << (4 * i);   // K padding stays zero
            }
            store_word(out, M, t, k0, word);
        }
    }
}

// One wave per row, for rows of at most 512 * CH values (K % 8 == 0).  The row is read through a
// row-sized buffer descriptor, so chunks past its end read as zero and neither the loads nor the
// quantizer need a branch; only the store of a chunk past the padded width is masked off.  RAGGED: any K and alignment.
template <int MODE, int CH, bool RAGGED>
__global__ __launch_bounds__(QT) void quantize_act_wave_kernel(const uint16_t *__restrict__ x, uint8_t *__restrict__ out, float *__restrict__ row_out,
                                                               const float *__restrict__ row_in, int64_t M, int Ki, float inv_s_a, int zoff_stream,
                                                               float eps)
{
    const int zoff = zoff_stream & 255, stream_in = zoff_stream & STREAM_IN;
    const int64_t K = Ki;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = (int64_t)blockIdx.x * (QT / 64) + wave;
    if (t >= M) return;
    const int Kpad = (int)(k_tiles(K) * KT);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(x + t * K), 0, Ki * 2, RSRC_FLAGS);

    q_v4u regs[CH];
    if (RAGGED) {
        load_row_chunks(regs, x + t * K, lane * QCHUNK, 64 * QCHUNK, Ki);
    } else if (stream_in) {
#pragma unroll
        for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * 64 + lane) * 16, 0, Q_STREAM);
    } else {
#pragma unroll
        for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * 64 + lane) * 16, 0, 0);
    }
    float r = 1.0f;
    if (MODE == FPTQ_SCALE_RMS) {
        double ss = 0.0;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double a = (double)bf16_to_f32(w[j] & 0xffffu), b = (double)bf16_to_f32(w[j] >> 16);
                ss = __builtin_fma(a, a, ss);
                ss = __builtin_fma(b, b, ss);
            }
        }
        ss = wave_sum(ss);
        r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    } else if (MODE == FPTQ_SCALE_GIVEN) {
        r = row_in[t];
    }
    const float c = (MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a;
    if (lane == 0 && row_out) row_out[t] = r;
    // chunk i of lane l is values 8 (64 i + l) ..: K tile 4 i + l / 16, byte 4 (l % 16) of the row's segment
    uint8_t *orow = out + (((int64_t)(lane >> 4) * M + t) * SEG + (lane & 15) * 4);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int k0 = (i * 64 + lane) * QCHUNK;
        const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
        uint32_t word = quant_chunk(w, c, zoff);
        word = RAGGED ? codes_inside(word, k0, Ki) : k0 >= Ki ? 0u : word;      // K padding stays zero
        if (k0 < Kpad) *reinterpret_cast<uint32_t *>(orow + (int64_t)(4 * i) * M * SEG) = word;
    }
}

// Dynamic quantization (App. B of the paper): the scale is computed at run time per token,
// s_t = max_k |x_t,k| / 7 (NaNs ignored; a zero or infinite maximum gives s_t = 1), then
// q = clamp(rne(x * (1 / s_t)), -8, 7).  One wave per row.  CH > 0: the row (K <= 512 * CH, K % 8 == 0 and 16-byte aligned unless RAGGED)
// stays in registers between the max reduction and the quantizer; CH == 0: any K, two passes.
__device__ inline uint32_t abs_bits_no_nan(uint32_t h)
{
    uint32_t m = h & 0x7fffu;
    return m > 0x7f80u ? 0u : m;       // bf16 magnitudes order like their bit patterns; NaN does not enter the max
}

template <int CH, bool RAGGED>
__global__ __launch_bounds__(QT) void quantize_act_dynamic_kernel(const uint16_t *__restrict__ x, int64_t M, int64_t K,
                                                                  uint8_t *__restrict__ out, float *__restrict__ s_out)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = (int64_t)blockIdx.x * (QT / 64) + wave;
    if (t >= M) return;
    const uint16_t *row = x + t * K;
    const int64_t Kpad = k_tiles(K) * KT;

    q_v4u regs[CH > 0 ? CH : 1];
    uint32_t mx = 0;
    if (CH > 0) {      // the row through a row-sized buffer descriptor: chunks past its end read as zero
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, (int)K * 2, RSRC_FLAGS);
        if (RAGGED) {
            load_row_chunks(regs, row, lane * QCHUNK, 64 * QCHUNK, (int)K);
        } else {
#pragma unroll
            for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * 64 + lane) * 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) mx = max(mx, max(abs_bits_no_nan(w[j] & 0xffffu), abs_bits_no_nan(w[j] >> 16)));
        }
    } else {
        for (int64_t k = lane; k < K; k += 64) mx = max(mx, abs_bits_no_nan(row[k]));
    }
    mx = wave_max(mx);
    const float amax = bf16_to_f32(mx);
    const float s = (amax > 0.0f && mx < 0x7f80u) ? amax / 7.0f : 1.0f;
    const float c = 1.0f / s;
    if (lane == 0) s_out[t] = s;

    if (CH > 0) {
        uint8_t *orow = out + (((int64_t)(lane >> 4) * M + t) * SEG + (lane & 15) * 4);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k0 = (i * 64 + lane) * QCHUNK;
            const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
            uint32_t word = quant_chunk(w, c, 8);
            word = RAGGED ? codes_inside(word, k0, (int)K) : k0 >= (int)K ? 0u : word;      // K padding stays zero
            if (k0 < (int)Kpad) *reinterpret_cast<uint32_t *>(orow + (int64_t)(4 * i) * M * SEG) = word;
        }
    } else {
        for (int64_t k0 = (int64_t)lane * QCHUNK; k0 < Kpad; k0 += 64 * QCHUNK) {
            uint32_t word = 0;
#pragma unroll
            for (int i = 0; i < QCHUNK; ++i) {
                int64_t k = k0 + i;
                if (k < K) word |= (quant_code(bf16_to_f32(row[k]), c, 8) ^ 8u) << (4 * i);
            }
            store_word(out, M, t, k0, word);
        }
    }
}

// The same with one workgroup per row (rows of at most 2048 * CH values; K % 8 == 0 and 16-byte aligned unless RAGGED): a row is
// spread over four waves, which is faster whenever rows are long or few.  RAGGED: 2048 x 4366 40 us by element in one wave, now 8.8, 279 x 11849 78 and 6.5.
template <int CH, bool RAGGED>
__global__ __launch_bounds__(QT) void quantize_act_dynamic_row_kernel(const uint16_t *__restrict__ x, int64_t M, int64_t K,
                                                                      uint8_t *__restrict__ out, float *__restrict__ s_out)
{
    __shared__ uint32_t red[QT / 64];
    const int64_t t = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t Kpad = k_tiles(K) * KT;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(x + t * K), 0, (int)K * 2, RSRC_FLAGS);
    q_v4u regs[CH];
    if (RAGGED) {
        load_row_chunks(regs, x + t * K, tid * QCHUNK, QT * QCHUNK, (int)K);
    } else {
#pragma unroll
        for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i * QT + tid) * 16, 0, 0);
    }
    uint32_t mx = 0;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) mx = max(mx, max(abs_bits_no_nan(w[j] & 0xffffu), abs_bits_no_nan(w[j] >> 16)));
    }
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < QT / 64; ++w) mx = max(mx, red[w]);
    const float amax = bf16_to_f32(mx);
    const float s = (amax > 0.0f && mx < 0x7f80u) ? amax / 7.0f : 1.0f;
    const float c = 1.0f / s;
    if (tid == 0) s_out[t] = s;
    uint8_t *orow = out + (((int64_t)(tid >> 4) * M + t) * SEG + (tid & 15) * 4);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int k0 = (i * QT + tid) * QCHUNK;
        const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
        uint32_t word = quant_chunk(w, c, 8);
        word = RAGGED ? codes_inside(word, k0, (int)K) : k0 >= (int)K ? 0u : word;      // K padding stays zero
        if (k0 < (int)Kpad) *reinterpret_cast<uint32_t *>(orow + (int64_t)(16 * i) * M * SEG) = word;
    }
}

hipError_t launch_quantize_act_dynamic(const uint16_t *x, int64_t M, int64_t K, uint8_t *out, float *s_out, hipStream_t s)
{
    const int64_t blocks = (M + QT / 64 - 1) / (QT / 64);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    dim3 grid((unsigned)blocks), block(QT);
    const bool vec = K % QCHUNK == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const int64_t Kpad = k_tiles(K) * KT;
    // Of 3073 to 4096 values as in the residual step, with other lines, as there is less to do per value.  2048 workgroups run at once: between one and a quarter and two
    // rounds of them the second costs more than the spreading gains (wave / workgroup, from HBM and from the cache: 1500 x 3584
    // 6.0 / 5.2, 4.5 / 4.2; 2560 x 3584 7.9 / 7.3, 6.0 / 5.9; 3000 x 3584 8.3 / 7.9, 6.4 / 6.8; 4096 x 3080 9.7 / 9.7, 7.6 / 8.4; 4096 x 3584 10.1 / 10.1, 8.0 / 8.7; 4096 x
    // 4096 11.0 / 10.6, 8.9 / 9.0; 6000 x 3584 13.3 / 13.1, 12.0 / 11.3; 8192 x 3080 15.9 / 16.6, 14.2 / 14.2; 8192 x 3584 17.2 / 17.6, 15.1 / 14.5; 16384 x 3840 31.2 / 31.2, 27.4 / 26.9;
    // 20000 x 3328 33.1 / 36, 29.9 / 31.1; 30000 x 3840 54.9 / 58.2, 46.3 / 53; 30000 x 4096 59.6 / 56.0, 53.6 / 54.9; 65536 x 4096 134.5 / 137.6, 134.6 / 138.6).
    if (wave_per_row(vec, M, K, M <= 2560 ? 3072 : M <= 4096 ? 3840 : M <= 16384 ? 3200 : M <= 32768 ? 3840 : 4096)) {
#define FPTQ_WAVE_CASE(CH, RAGGED) quantize_act_dynamic_kernel<CH, RAGGED><<<grid, block, 0, s>>>(x, M, K, out, s_out)
        WAVE_PER_ROW(vec, Kpad, FPTQ_WAVE_CASE);
#undef FPTQ_WAVE_CASE
        return hipGetLastError();
    }
    if (M > 0x7fffffff) return hipErrorInvalidValue;
#define FPTQ_DYN_CASE(CH)                                                                          \
    if (vec && Kpad <= 2048 * CH) {                                                                \
        quantize_act_dynamic_row_kernel<CH, false><<<dim3((unsigned)M), block, 0, s>>>(x, M, K, out, s_out); \
        return hipGetLastError();                                                                  \
    }
    FPTQ_DYN_CASE(1)
    FPTQ_DYN_CASE(2)
    FPTQ_DYN_CASE(4)
    FPTQ_DYN_CASE(6)
    FPTQ_DYN_CASE(7)
    FPTQ_DYN_CASE(8)
    FPTQ_DYN_CASE(12)
    FPTQ_DYN_CASE(14)
    FPTQ_DYN_CASE(16)
#undef FPTQ_DYN_CASE
#define FPTQ_RAGGED_CASE(CH)                                                                       \
    if (Kpad <= 2048 * CH) {                                                                       \
        quantize_act_dynamic_row_kernel<CH, true><<<dim3((unsigned)M), block, 0, s>>>(x, M, K, out, s_out); \
        return hipGetLastError();                                                                  \
    }
    FPTQ_RAGGED_CASE(1)
    FPTQ_RAGGED_CASE(2)
    FPTQ_RAGGED_CASE(4)
    FPTQ_RAGGED_CASE(8)
    FPTQ_RAGGED_CASE(16)
#undef FPTQ_RAGGED_CASE
    quantize_act_dynamic_kernel<0, false><<<grid, block, 0, s>>>(x, M, K, out, s_out);
    return hipGetLastError();
}

// Scale given or none, aligned rows: a wave takes 512 CH consecutive values, consecutive waves consecutive pieces, and no wave waits for another.
// Bound by memory (us, a workgroup or wave per row before / now; inputs from HBM, in brackets from the last-level cache): 4096 x 14336 33.1 / 29.0 (24.1 /
// 24.0), 4096 x 11008 26.4 / 23.1 (18.7 / 18.2), 8192 x 8192 37.9 / 34.2 (25.9 / 26.9), 4096 x 4096 10.4 / 9.7 (7.6 / 7.1), 8192 x 28672 117.1 / 104.4; 64 x 13824
// 3.20 / 2.49, 1 x 13824 2.63 / 2.23, 1 x 4096 2.11 / 2.10.
template <int MODE, int CH, bool STREAM>
__global__ __launch_bounds__(QT) void quantize_act_flat_kernel(const uint16_t *__restrict__ x, uint8_t *__restrict__ out, float *__restrict__ row_out,
                                                               const float *__restrict__ row_in, int M, int K, float inv_s_a, int zoff, uint32_t pieces,
                                                               uint32_t per_pieces)
{
    static_assert(MODE != FPTQ_SCALE_RMS, "that scale takes the whole row");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t t, piece;
    divide(blockIdx.x * (QT / 64) + wave, pieces, per_pieces, t, piece);
    if (t >= (uint32_t)M) return;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(x + (int64_t)t * K), 0, K * 2, RSRC_FLAGS);
    const int k0 = (int)piece * (512 * CH) + lane * QCHUNK;
    q_v4u regs[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) regs[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (k0 + i * 512) * 2, 0, STREAM ? Q_STREAM : 0);
    const float r = MODE == FPTQ_SCALE_GIVEN ? row_in[t] : 1.0f;
    const float c = MODE == FPTQ_SCALE_NONE ? inv_s_a : r * inv_s_a;
    if (lane == 0 && piece == 0 && row_out) row_out[t] = r;
    // chunk i of lane l is values k0 + 512 i ..: K tile 4 (CH piece + i) + l / 16, byte 4 (l % 16) of the row's segment
    uint8_t *orow = out + (((int64_t)(piece * (4 * CH) + (lane >> 4)) * M + t) * SEG + (lane & 15) * 4);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int k = k0 + i * 512;
        const uint32_t w[4] = {regs[i].x, regs[i].y, regs[i].z, regs[i].w};
        const uint32_t word = quant_chunk(w, c, zoff);
        if (k < (K + KT - 1) / KT * KT) *reinterpret_cast<uint32_t *>(orow + (int64_t)(4 * i) * M * SEG) = k >= K ? 0u : word;      // K padding stays zero
    }
}

// Chunks a lane.  One below 16 MB, where larger pieces would leave waves' places empty (768 x 4096 3.1 us, four chunks 3.8), and for rows of up to 512 values.
// Other short rows are a piece each: cut by 512 values, their last piece is mostly padding (85481 x 1104 55.2 us, in one piece 48.3; 45900 x 2056 51.4 and 44.7, from the
// cache 24320 x 2048 39.0 and 36.0), and chunks that lie past a row's end are computed all the same (40000 x 256 in pieces of four 15.0 us, of one 9.9; 524288 x 512 170
// and 126; 97280 x 1024 in pieces of four 46.3, of two 44.2).  Longer rows, up to 40 MB, which four chunks a lane bring to the CUs in one round or little more: four (4096 x
// 4096 9.8 us, one 10.05, from the cache 7.1 and 8.3), but not where a sixteenth or more is padding (1700 x 11008 11.7, one 10.6); beyond, one (4096 x
// 14336 29.0, four 30.1), but not where so much is padding with one (19660 x 3200 33.1, four 30.8; 22995 x 4104 49.4, six 47.3).  More than the last-level cache holds:
// streaming loads, four chunks (8192 x 28672 102 us, one 110, without streaming 113 to 124).
static int flat_chunks(int64_t M, int64_t K)
{
    const int64_t mb = M * K * 2 >> 20;
    auto little_padding = [&](int64_t piece) { return (K + piece - 1) / piece * piece * 16 <= K * 17; };
    if (mb < 16 || K <= 512) return 1;
    if (K <= 3072) return K <= 1024 ? 2 : K <= 2048 ? 4 : 6;
    if (M * K * 2 > ((int64_t)256 << 20)) return K <= 4096 ? 8 : 4;
    if (mb < 40) return K <= 4096 || little_padding(2048) ? 4 : 1;
    return little_padding(512) ? 1 : K <= 4096 ? 4 : 6;
}
static int64_t flat_pieces(int64_t M, int64_t K) { return (K + 512 * flat_chunks(M, K) - 1) / (512 * flat_chunks(M, K)); }

template <int MODE>
static hipError_t launch_flat(const uint16_t *x, int64_t M, int64_t K, const float *row_in, float inv_s_a, int zoff, uint8_t *out, float *row_out, hipStream_t s)
{
    const bool stream = M * K * 2 > ((int64_t)256 << 20);
    const int64_t pieces = flat_pieces(M, K);
    const dim3 grid((unsigned)((M * pieces + QT / 64 - 1) / (QT / 64))), block(QT);
#define FPTQ_FLAT(CH, STREAM) quantize_act_flat_kernel<MODE, CH, STREAM><<<grid, block, 0, s>>>(x, out, row_out, row_in, (int)M, (int)K, inv_s_a, zoff, (uint32_t)pieces, reciprocal((uint32_t)pieces))
#define FPTQ_FLAT_CASE(CH)                    \
    case CH:                                  \
        if (stream) FPTQ_FLAT(CH, true);      \
        else FPTQ_FLAT(CH, false);            \
        break
    switch (flat_chunks(M, K)) {
        FPTQ_FLAT_CASE(1);
        FPTQ_FLAT_CASE(2);
        FPTQ_FLAT_CASE(4);
        FPTQ_FLAT_CASE(6);
    default: FPTQ_FLAT(8, true);
    }
#undef FPTQ_FLAT_CASE
#undef FPTQ_FLAT
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_mode(const uint16_t *x, int64_t M, int64_t K, float eps, const float *row_in, float inv_s_a,
                              int zoff, uint8_t *out, float *row_out, hipStream_t s)
{
    dim3 grid((unsigned)M), block(QT);
    const bool vec = K % QCHUNK == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const int64_t Kpad = k_tiles(K) * KT;
    dim3 wgrid((unsigned)((M + QT / 64 - 1) / (QT / 64)));
#define FPTQ_WAVE_CASE(CH, RAGGED) quantize_act_wave_kernel<MODE, CH, RAGGED><<<wgrid, block, 0, s>>>(x, out, row_out, row_in, M, (int)K, inv_s_a, zoff | stream_in, eps)
#define FPTQ_ROW_CASE(CH, RAGGED)                                                                                           \
    if (Kpad <= 2048 * CH) {                                                                                                \
        quantize_act_kernel<MODE, CH, RAGGED><<<grid, block, 0, s>>>(x, out, row_out, row_in, M, (int)K, inv_s_a, zoff | stream_in, eps); \
        return hipGetLastError();                                                                                           \
    }
    if constexpr (MODE != FPTQ_SCALE_RMS) {
        if (vec && K <= (1 << 28) && M * flat_pieces(M, K) <= MAX_WAVES) return launch_flat<MODE>(x, M, K, row_in, inv_s_a, zoff, out, row_out, s);
    } else if (vec) {
        // An input that the 256 MB last-level cache cannot hold is read with streaming loads (8192 x 28672: 119 us
        // against 142); a smaller one is usually still there from its producer, and ordinary loads are faster on it.
        const int stream_in = M * K * 2 > ((int64_t)256 << 20) ? STREAM_IN : 0;
        // A workgroup per row, which spreads a row over four waves (32 x 11008: 2.9 us against 5.6; 2048 x 11008: 10.8 against 12.9), but for
        // short rows in large numbers (2048 x 4096 the other way, 6.0 against 5.3).
        if (wave_per_row(true, M, K)) {
            if (Kpad <= 2048) FPTQ_WAVE_CASE(4, false);
            else FPTQ_WAVE_CASE(8, false);
            return hipGetLastError();
        }
        // chunks per thread: 6 covers the Llama-2 FFN width 11008, 7 and 14 are the Llama-3 FFN widths 14336 and 28672
        FPTQ_ROW_CASE(1, false)
        FPTQ_ROW_CASE(2, false)
        FPTQ_ROW_CASE(4, false)
        FPTQ_ROW_CASE(6, false)
        FPTQ_ROW_CASE(7, false)
        FPTQ_ROW_CASE(8, false)
        FPTQ_ROW_CASE(12, false)
        FPTQ_ROW_CASE(14, false)
        FPTQ_ROW_CASE(16, false)
    }
    constexpr int stream_in = 0;
    if (!vec || MODE != FPTQ_SCALE_RMS) {
        if (wave_per_row(false, M, K)) {
            WAVE_PER_ROW_RAGGED(Kpad, FPTQ_WAVE_CASE);
            return hipGetLastError();
        }
        FPTQ_ROW_CASE(1, true)
        FPTQ_ROW_CASE(2, true)
        FPTQ_ROW_CASE(4, true)
        FPTQ_ROW_CASE(8, true)
        FPTQ_ROW_CASE(16, true)
    }
#undef FPTQ_WAVE_CASE
#undef FPTQ_ROW_CASE
    quantize_act_kernel<MODE, 0, false><<<grid, block, 0, s>>>(x, out, row_out, row_in, M, K, inv_s_a, zoff, eps);
    return hipGetLastError();
}

hipError_t launch_quantize_act(const uint16_t *x, int64_t M, int64_t K, int mode, float eps, const float *row_in,
                               float inv_s_a, int zero_point, uint8_t *out, float *row_out, hipStream_t s)
{
    if (M > 0x7fffffff) return hipErrorInvalidValue;
    switch (mode) {
    case FPTQ_SCALE_NONE: return launch_mode<FPTQ_SCALE_NONE>(x, M, K, eps, row_in, inv_s_a, zero_point + 8, out, row_out, s);
    case FPTQ_SCALE_RMS: return launch_mode<FPTQ_SCALE_RMS>(x, M, K, eps, row_in, inv_s_a, zero_point + 8, out, row_out, s);
    default: return launch_mode<FPTQ_SCALE_GIVEN>(x, M, K, eps, row_in, inv_s_a, zero_point + 8, out, row_out, s);
    }
}

}  // namespace fptq
