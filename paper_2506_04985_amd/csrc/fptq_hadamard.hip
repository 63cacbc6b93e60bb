// Online Hadamard transform in front of the down projection (Sec. 3.1.4 and App. D, "Hadamard
// non-powers of 2" of the paper), fused with the per-token scale, the static INT4 quantizer and
// the packer: x -> clamp(rne((x H_B / sqrt(B)) * S_t / s_a), -8, 7), block-wise over consecutive
// groups of B channels (B = 256, 512, 1024, 2048 or 4096: the largest power of two dividing the
// down projection's width is 256 for 11008, 2048 for 14336, 4096 for 28672), one pass over X.
//
// The transform is evaluated by the in-place butterfly network in fp32 with strides
// 128, 64, ..., 1, each pair (a, b) -> (a + b, a - b): every output is a fixed tree of fp32
// additions, so the result does not depend on how the work is spread over lanes.
//
// B = 256.  One wave per token row; a wave walks the row in super-chunks of 1024 values = 4 blocks, a
// block per 16 lanes, 16 values per lane.  The four high strides need the lane to hold
// x[16 j + g] (j = 0..15), the four low strides x[16 g + e]: the bf16 values are loaded in the strided view (16 loads side by side;
// through LDS, as whole lines, was 2 to 4 % slower), the fp32 intermediates go through LDS to get the contiguous view
// (padded so that both directions are bank-conflict free).  Everything is wave-private: no barriers.
//
// Bound by HBM (2 bytes read, half a byte written per value) and VALU issue: 16 VALU instructions per value at B = 256, 21 at B = 2048
// and 4096 with a workgroup per block, 20 with a wave per block, which keep the SIMDs issuing in 62 % of all cycles at 4096 x 11008,
// 88 % at 4096 x 14336 and 90 % at 8192 x 28672 (the plain quantizer: 33 to 39 %).  4096 x 11008 takes 26.7 us (27.3 before the loads were direct).
//
// B = 64 V with V = 8, 16, 32, 64 (32 and 64: in RMS mode, and beyond the number of blocks at which a workgroup per block is the faster).  One block per wave iteration, V values per lane.  View 1: the lane
// holds x[64 j + lane] and runs strides B/2 .. 64 in registers; view 2: the lane holds
// x[V lane + e] and runs strides V/2 .. 1 in registers; the strides in between (32 .. V) pair lane l with
// lane l ^ (stride / V) and are done with DPP lane exchanges, in descending order between the two
// register passes, so the stage order is that of the definition.  The raw block and the fp32
// transposition patch share the wave's LDS region (a wave's LDS operations complete in order).
#include "fptq_common.h"

namespace fptq {

constexpr int HB = 256;                 // Hadamard block
constexpr int H_F32_ROW = 20;           // words per 16-value row of the fp32 transpose patch (16 + 4)
constexpr int H_F32_BLK = 336;          // words per block of the patch (16 * 20 + 16)
// 5376 bytes of patch, rounded up so that five workgroups share a CU: a line is loaded by four instructions, and the lines in flight of seven
// workgroups do not fit L1 (8192 x 13824: 64.3 us with seven, 60.2 with five)
constexpr int H_WAVE_LDS = 7552;
static_assert(H_WAVE_LDS >= 4 * H_F32_BLK * 4, "");

__device__ inline float h_bf16_to_f32(uint32_t bits) { return __uint_as_float(bits << 16); }

__device__ inline void butterflies16(float (&v)[16])
{
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if ((j & s) == 0) {
                float a = v[j], b = v[j + s];
                v[j] = a + b;
                v[j + s] = a - b;
            }
}

template <int MODE>
__global__ __launch_bounds__(256) void quantize_act_hadamard_kernel(const uint16_t *__restrict__ x, int64_t M, int64_t K,
                                                                    float eps, const float *__restrict__ row_in,
                                                                    float inv_s_a, float hnorm, uint8_t *__restrict__ out,
                                                                    float *__restrict__ row_out, int ksplit)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[4 * H_WAVE_LDS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // ksplit waves share a row: wave `part` of them takes every ksplit-th group of four blocks
    const int64_t wid = (int64_t)blockIdx.x * 4 + wave, t = wid / ksplit;
    const int part = (int)(wid % ksplit);
    if (t >= M) return;                                  // whole waves leave; nothing below synchronises
    const uint16_t *row = x + t * K;

    float r = 1.0f;
    if (MODE == FPTQ_SCALE_RMS) {                        // S_t from the row as the norm layer sees it
        double ss = 0.0;
        for (int64_t k0 = (int64_t)lane * 8; k0 < K; k0 += 512) {
            const uint4 u = *reinterpret_cast<const uint4 *>(row + k0);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double a = (double)h_bf16_to_f32(w[j] & 0xffffu), b = (double)h_bf16_to_f32(w[j] >> 16);
                ss = __builtin_fma(a, a, ss);
                ss = __builtin_fma(b, b, ss);
            }
        }
        ss = wave_sum(ss);
        r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    } else if (MODE == FPTQ_SCALE_GIVEN) {
        r = row_in[t];
    }
    const float c = ((MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a) * hnorm;
    if (lane == 0 && part == 0 && row_out) row_out[t] = r;

    const int b = lane >> 4, g = lane & 15;
    // a lane's 16 results: K tile 2 b + g / 8 of the super-chunk's, bytes 8 (g % 8) of the row's segment
    const int64_t lane_out = (int64_t)(2 * b + (g >> 3)) * M * SEG + (g & 7) * 8;
    float *patch = reinterpret_cast<float *>(lds + wave * H_WAVE_LDS) + b * H_F32_BLK;

    for (int64_t sc = (int64_t)part * (4 * HB); sc < K; sc += (int64_t)ksplit * (4 * HB)) {
        const int live_blocks = (int)min((int64_t)4, (K - sc) / HB);      // lanes of blocks past the row's end repeat the last one
        // strided view x[16 j + g]: strides 128, 64, 32, 16 of the block are strides 8, 4, 2, 1 in j
        float v[16];
        const uint16_t *const src = row + sc;
        const int at = min(b, live_blocks - 1) * HB + g;
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = h_bf16_to_f32(src[at + 16 * j]);
        butterflies16(v);
        // transpose inside the block: value (j, g) to row j, column g; read back row g
#pragma unroll
        for (int j = 0; j < 16; ++j) patch[H_F32_ROW * j + g] = v[j];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 f = *reinterpret_cast<const float4 *>(patch + H_F32_ROW * g + 4 * i);
            v[4 * i] = f.x, v[4 * i + 1] = f.y, v[4 * i + 2] = f.z, v[4 * i + 3] = f.w;
        }
        butterflies16(v);                                 // contiguous view: strides 8, 4, 2, 1
        if (b < live_blocks) {
            uint32_t w0 = 0, w1 = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                w0 |= quant_code(v[e], c, 8) << (4 * e);
                w1 |= quant_code(v[8 + e], c, 8) << (4 * e);
            }
            w0 ^= CODE_TO_NIBBLES, w1 ^= CODE_TO_NIBBLES;
            *reinterpret_cast<uint2 *>(out + ((sc / KT) * M + t) * SEG + lane_out) = make_uint2(w0, w1);
        }
    }
}


// ---------------------------------------------------------------------------------- B = 512 .. 4096
template <int V>
__device__ inline void butterflies(float (&v)[V])
{
#pragma unroll
    for (int s = V / 2; s >= 1; s >>= 1)
#pragma unroll
        for (int j = 0; j < V; ++j)
            if ((j & s) == 0) {
                float a = v[j], b = v[j + s];
                v[j] = a + b;
                v[j + s] = a - b;
            }
}

// value of lane (l ^ MASK), MASK = 1, 2 (DPP quad permutation) or 4 (swizzle within 32 lanes)
template <int MASK>
__device__ inline float lane_xor(float x)
{
    const int i = __float_as_int(x);
    if (MASK == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    if (MASK == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    return __int_as_float(__builtin_amdgcn_ds_swizzle(i, 0x101F));                                   // and 0x1f, xor 4
}

// one butterfly stage across lanes: the lower lane of a pair gets a + b, the upper one a - b, where a
// is the lower lane's value: both are other + (upper ? -own : own), and negation is exact
template <int MASK, int V>
__device__ inline void cross_stage(float (&v)[V], int lane)
{
    const uint32_t flip = (lane & MASK) ? 0x80000000u : 0u;
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = lane_xor<MASK>(v[e]) + __uint_as_float(__float_as_uint(v[e]) ^ flip);
}

template <int MODE, int V>
__global__ __launch_bounds__(256) void quantize_act_hadamard_wide_kernel(const uint16_t *__restrict__ x, int64_t M, int64_t K,
                                                                         float eps, const float *__restrict__ row_in,
                                                                         float inv_s_a, float hnorm, uint8_t *__restrict__ out,
                                                                         float *__restrict__ row_out, int ksplit)
{
    constexpr int B = 64 * V;
    constexpr int WAVE_WORDS = B + 256;          // fp32 patch: 4 pad words after every V elements (64 groups)
    extern __shared__ __attribute__((aligned(16))) uint8_t wide_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t wid = (int64_t)blockIdx.x * 4 + wave, t = wid / ksplit;     // ksplit waves share a row, block by block
    const int part = (int)(wid % ksplit);
    if (t >= M) return;                                  // whole waves leave; nothing below synchronises
    const uint16_t *row = x + t * K;

    float r = 1.0f;
    if (MODE == FPTQ_SCALE_RMS) {                        // S_t from the row as the norm layer sees it
        double ss = 0.0;
        for (int64_t k0 = (int64_t)lane * 8; k0 < K; k0 += 512) {
            const uint4 u = *reinterpret_cast<const uint4 *>(row + k0);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double a = (double)h_bf16_to_f32(w[j] & 0xffffu), b = (double)h_bf16_to_f32(w[j] >> 16);
                ss = __builtin_fma(a, a, ss);
                ss = __builtin_fma(b, b, ss);
            }
        }
        ss = wave_sum(ss);
        r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    } else if (MODE == FPTQ_SCALE_GIVEN) {
        r = row_in[t];
    }
    const float c = ((MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a) * hnorm;
    if (lane == 0 && part == 0 && row_out) row_out[t] = r;

    uint8_t *raw = wide_lds + wave * (WAVE_WORDS * 4);
    float *patch = reinterpret_cast<float *>(raw);

    for (int64_t sc = (int64_t)part * B; sc < K; sc += (int64_t)ksplit * B) {
        // linear copy of the block into LDS, 1 KB per wave-level load
#pragma unroll
        for (int i = 0; i < V / 8; ++i)
            *reinterpret_cast<uint4 *>(raw + (i * 64 + lane) * 16) = *reinterpret_cast<const uint4 *>(row + sc + (i * 64 + lane) * 8);
        float v[V];
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = h_bf16_to_f32(*reinterpret_cast<const uint16_t *>(raw + (64 * j + lane) * 2));
        butterflies<V>(v);                                // strides B/2 .. 64
        // element e = 64 j + lane goes to word e + 4 (e / V); the lane then reads its V contiguous elements
#pragma unroll
        for (int j = 0; j < V; ++j) patch[j * (64 + 256 / V) + lane + 4 * (lane / V)] = v[j];
#pragma unroll
        for (int i = 0; i < V / 4; ++i) {
            const float4 f = *reinterpret_cast<const float4 *>(patch + lane * (V + 4) + 4 * i);
            v[4 * i] = f.x, v[4 * i + 1] = f.y, v[4 * i + 2] = f.z, v[4 * i + 3] = f.w;
        }
        if (V <= 8) cross_stage<4, V>(v, lane);           // stride 32 at V = 8
        if (V <= 16) cross_stage<2, V>(v, lane);          // stride 32 at V = 16, stride 16 at V = 8
        if (V <= 32) cross_stage<1, V>(v, lane);          // stride V
        butterflies<V>(v);                                // strides V/2 .. 1
        uint32_t w[V / 8];
#pragma unroll
        for (int i = 0; i < V / 8; ++i) {
            w[i] = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) w[i] |= quant_code(v[8 * i + e], c, 8) << (4 * e);
            w[i] ^= CODE_TO_NIBBLES;
        }
        const int64_t k0 = sc + (int64_t)V * lane;        // V <= 128 values never straddle a K tile
        uint8_t *dst = out + ((k0 / KT) * M + t) * SEG + (k0 % KT) / 2;
        if (V == 8) *reinterpret_cast<uint32_t *>(dst) = w[0];
        if (V == 16) *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
        if (V >= 32) {
#pragma unroll
            for (int i = 0; i < V / 32; ++i)
                *reinterpret_cast<uint4 *>(dst + 16 * i) = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
        }
    }
}

// ---------------------------------------------------------------------------------- B = 2048, 4096, few blocks
// A workgroup of B / 16 threads per block, 16 values a thread: where the whole call is the latency of one block, a wave that holds all of it
// takes four times as many instructions one after the other (one token of 14336 values 3.4 us, now 2.7, 28672 4.8 and 2.8).  Three views of the
// block, elements e of LOGB bits: thread = the low bits, registers = the top four (loaded as they are: 16 loads side by side); registers =
// the next four, thread = the rest; 16 consecutive elements a thread.  The strides run from B / 2 to 1 as in the definition, four
// (in the last view of B = 2048 three) per view.  Between views the values go through LDS, the first time across waves (a barrier), the second
// inside the thread's wave; element e lies in word e + 4 (e / 16) + 2^(LOGB-8) (e / 2^(LOGB-4)), which leaves the second view free of bank conflicts, and
// the third one's reads for B = 4096.  For B = 2048 threads t and t + 6 of 16 meet there, and in the first view's stores lanes 52 to 63 of a wave meet 0 to 11:
// 64 conflict cycles a wave counted at 4096 x 14336.
template <int MODE, int LOGB>
__global__ __launch_bounds__(1 << (LOGB - 4)) void quantize_act_hadamard_group_kernel(const uint16_t *__restrict__ x, int64_t M, int64_t K,
                                                                                     const float *__restrict__ row_in, float inv_s_a, float hnorm,
                                                                                     uint8_t *__restrict__ out, float *__restrict__ row_out, int blocks)
{
    static_assert(LOGB == 11 || LOGB == 12, "views of four bits");
    constexpr int B = 1 << LOGB, THREADS = B / 16, LOW = LOGB - 8;      // LOW bits below the second view's four
    __shared__ __attribute__((aligned(16))) float lds[B + B / 4 + (16 << LOW)];
    auto word = [](int e) { return e + 4 * (e >> 4) + ((e >> (LOGB - 4)) << LOW); };
    const int t = threadIdx.x;
    const int64_t m = blockIdx.x / blocks;
    const int blk = (int)(blockIdx.x % blocks);
    const uint16_t *row = x + m * K, *src = row + (int64_t)blk * B;
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = h_bf16_to_f32(src[j * THREADS + t]);

    float r = 1.0f;
    if (MODE == FPTQ_SCALE_GIVEN) r = row_in[m];
    const float c = ((MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a) * hnorm;
    if (t == 0 && blk == 0 && row_out) row_out[m] = r;

    butterflies16(v);
    // word() of a thread's element plus that of a register's: no bit of one carries into the other
    float *const first = lds + t + 4 * (t >> 4), *const second = lds + word(((t >> LOW) << (LOGB - 4)) | (t & ((1 << LOW) - 1)));
#pragma unroll
    for (int j = 0; j < 16; ++j) first[word(j * THREADS)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = second[word(j << LOW)];
    butterflies16(v);
    // a thread writes the elements it has read; the ones it reads next were written by its own wave, whose LDS operations complete in order
#pragma unroll
    for (int j = 0; j < 16; ++j) second[word(j << LOW)] = v[j];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 f = *reinterpret_cast<const float4 *>(lds + word(t * 16) + 4 * i);
        v[4 * i] = f.x, v[4 * i + 1] = f.y, v[4 * i + 2] = f.z, v[4 * i + 3] = f.w;
    }
#pragma unroll
    for (int s = LOGB == 12 ? 8 : 4; s >= 1; s >>= 1)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if ((j & s) == 0) {
                const float a = v[j], b = v[j + s];
                v[j] = a + b;
                v[j + s] = a - b;
            }
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e / 8] |= quant_code(v[e], c, 8) << (4 * (e % 8));
    const int64_t k0 = (int64_t)blk * B + t * 16;
    *reinterpret_cast<uint2 *>(out + ((k0 / KT) * M + m) * SEG + (k0 % KT) / 2) = make_uint2(w[0] ^ CODE_TO_NIBBLES, w[1] ^ CODE_TO_NIBBLES);
}

template <int LOGB>
static hipError_t launch_group(const uint16_t *x, int64_t M, int64_t K, int mode, const float *row_in, float inv_s_a, uint8_t *out,
                               float *row_out, hipStream_t s)
{
    const int blocks = (int)(K >> LOGB);
    const float hnorm = (float)(1.0 / sqrt((double)(1 << LOGB)));
    dim3 grid((unsigned)(M * blocks)), block(1 << (LOGB - 4));
    if (mode == FPTQ_SCALE_GIVEN)
        quantize_act_hadamard_group_kernel<FPTQ_SCALE_GIVEN, LOGB><<<grid, block, 0, s>>>(x, M, K, row_in, inv_s_a, hnorm, out, row_out, blocks);
    else
        quantize_act_hadamard_group_kernel<FPTQ_SCALE_NONE, LOGB><<<grid, block, 0, s>>>(x, M, K, row_in, inv_s_a, hnorm, out, row_out, blocks);
    return hipGetLastError();
}

// Waves per row: with few rows a wave per row leaves the device idle (one token of 11008 values took 9.5 us, as
// long as 512 tokens), so the blocks of a row are dealt to as many waves as it takes to have about 4096 in all
// (16384 was slower again: 2048 x 11008 17.1 us against 13.9).
// In RMS mode every wave of a row sums the whole row again, which only pays while there are few rows.
static int waves_per_row(int64_t M, int64_t chunks, int mode)
{
    if (M >= 4096 || (mode == FPTQ_SCALE_RMS && M > 256)) return 1;
    const int64_t want = (4096 + M - 1) / M;
    return (int)(want < chunks ? want : chunks);
}

constexpr int wide_lds_bytes(int v) { return 4 * (64 * v + 256) * 4; }

template <int MODE, int V>
static hipError_t set_wide_attribute()
{
    if (wide_lds_bytes(V) <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void *)quantize_act_hadamard_wide_kernel<MODE, V>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               wide_lds_bytes(V));
}

// Once per device: more than 64 KB of dynamic LDS has to be asked for before the first launch.
hipError_t hadamard_device_init(int)
{
    hipError_t e = hipSuccess;
    auto one = [&](hipError_t r) { if (e == hipSuccess) e = r; };
#define FPTQ_WIDE_ATTR(V) one(set_wide_attribute<FPTQ_SCALE_NONE, V>()), one(set_wide_attribute<FPTQ_SCALE_RMS, V>()), one(set_wide_attribute<FPTQ_SCALE_GIVEN, V>())
    FPTQ_WIDE_ATTR(8);
    FPTQ_WIDE_ATTR(16);
    FPTQ_WIDE_ATTR(32);
    FPTQ_WIDE_ATTR(64);
#undef FPTQ_WIDE_ATTR
    return e;
}

template <int V>
static hipError_t launch_wide(const uint16_t *x, int64_t M, int64_t K, int mode, float eps, const float *row_in, float inv_s_a,
                              uint8_t *out, float *row_out, hipStream_t s)
{
    const int ksplit = waves_per_row(M, (K + 64 * V - 1) / (64 * V), mode);
    const int64_t blocks = (M * ksplit + 3) / 4;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    constexpr int LDS_BYTES = wide_lds_bytes(V);
    const DeviceInfo *info;
    hipError_t e0 = device_info(&info);       // the kernels that need more than 64 KB of dynamic LDS got their limit there
    if (e0 != hipSuccess) return e0;
    const float hnorm = (float)(1.0 / sqrt((double)(64 * V)));
    dim3 grid((unsigned)blocks), block(256);
#define FPTQ_LAUNCH_WIDE(MODE)                                                                                             \
    do {                                                                                                                   \
        auto kern = quantize_act_hadamard_wide_kernel<MODE, V>;                                                            \
        kern<<<grid, block, LDS_BYTES, s>>>(x, M, K, eps, row_in, inv_s_a, hnorm, out, row_out, ksplit);                   \
    } while (0)
    switch (mode) {
    case FPTQ_SCALE_NONE: FPTQ_LAUNCH_WIDE(FPTQ_SCALE_NONE); break;
    case FPTQ_SCALE_RMS: FPTQ_LAUNCH_WIDE(FPTQ_SCALE_RMS); break;
    default: FPTQ_LAUNCH_WIDE(FPTQ_SCALE_GIVEN);
    }
#undef FPTQ_LAUNCH_WIDE
    return hipGetLastError();
}

hipError_t launch_quantize_act_hadamard(const uint16_t *x, int64_t M, int64_t K, int hadamard_block, int mode, float eps,
                                        const float *row_in, float inv_s_a, uint8_t *out, float *row_out, hipStream_t s)
{
    // A workgroup per block, unless its scale would have to be summed in every wave of every block, over the whole row (RMS mode: 1 x 14336
    // 8.5 -> 7.4 us, but 16 x 14336 10.6 -> 11.5, 2048 x 28672 64 -> 223)
    // and up to 32768 blocks (4096 x 14336 35.4 -> 34.3, 2048 x 28672 42.0 -> 36.2, 4096 x 8192 25.2 -> 21.5; 8192 x 14336 66.6, 67.4)
    if (hadamard_block >= 2048 && mode != FPTQ_SCALE_RMS && M <= 32768 && M * (K / hadamard_block) <= 32768)
        return hadamard_block == 2048 ? launch_group<11>(x, M, K, mode, row_in, inv_s_a, out, row_out, s)
                                      : launch_group<12>(x, M, K, mode, row_in, inv_s_a, out, row_out, s);
    switch (hadamard_block) {
    case 512: return launch_wide<8>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 1024: return launch_wide<16>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 2048: return launch_wide<32>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 4096: return launch_wide<64>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 256: break;
    default: return hipErrorInvalidValue;
    }
    const int ksplit = waves_per_row(M, (K + 4 * HB - 1) / (4 * HB), mode);
    const int64_t blocks = (M * ksplit + 3) / 4;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const float hnorm = 1.0f / 16.0f;       // 1 / sqrt(256)
    dim3 grid((unsigned)blocks), block(256);
    switch (mode) {
    case FPTQ_SCALE_NONE:
        quantize_act_hadamard_kernel<FPTQ_SCALE_NONE><<<grid, block, 0, s>>>(x, M, K, eps, row_in, inv_s_a, hnorm, out, row_out, ksplit);
        break;
    case FPTQ_SCALE_RMS:
        quantize_act_hadamard_kernel<FPTQ_SCALE_RMS><<<grid, block, 0, s>>>(x, M, K, eps, row_in, inv_s_a, hnorm, out, row_out, ksplit);
        break;
    default:
        quantize_act_hadamard_kernel<FPTQ_SCALE_GIVEN><<<grid, block, 0, s>>>(x, M, K, eps, row_in, inv_s_a, hnorm, out, row_out, ksplit);
    }
    return hipGetLastError();
}

}  // namespace fptq
