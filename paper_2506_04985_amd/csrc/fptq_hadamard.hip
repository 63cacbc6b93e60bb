// Online Hadamard transform in front of the down projection (Sec. 3.1.4 and App. D, "Hadamard
// non-powers of 2" of the paper), fused with the per-token scale, the static INT4 quantizer and
// the packer: x -> clamp(rne((x H_B / sqrt(B)) * S_t / s_a), -8, 7), block-wise over consecutive
// groups of B channels (B = 256, 512, 1024, 2048 or 4096: the largest power of two dividing the
// down projection's width is 256 for 11008, 2048 for 14336, 4096 for 28672), one pass over X.
//
// The transform is evaluated by the in-place butterfly network in fp32 with strides
// B / 2, B / 4, ..., 1, each pair (a, b) -> (a + b, a - b): every output is a fixed tree of fp32
// additions, so the result does not depend on how the work is spread over lanes.
//
// A wave holds 1024 consecutive values of a row (a block of 2048 or 4096) in registers from the load to the codes, without LDS: the first
// strides run over registers, then over lanes, then over registers again.  Where the scale is given, every wave is done after one such
// span, consecutive waves take consecutive spans, and memory is read in the order it lies in; waves that walked a row each, or several spans
// a row apart, were up to a sixth slower on inputs that come from HBM (us, the kernel that walked rows through LDS and this one):
//     4096 x 11008, B = 256    28.8  24.4     4096 x 13824, B = 512   40.7  30.7     4096 x 11264, B = 1024   30.8  27.3
//     8192 x 14336, B = 2048   70.2  66.2     8192 x 13824, B = 512   72.0  61.2     8192 x 28672, B = 4096  137.0 121.0
// (one card; the read alone, as one burst: 16.3 us at 4096 x 11008, 80.6 at 8192 x 28672; from the last-level cache 4096 x 11008 22.1 and 21.8).
// Bound by memory there and by VALU issue from the cache: 17.5 instructions per value counted at B = 256, 18.6 at 512, 19.1 at 1024, 18.8 at 2048
// and 19.1 at 4096, a wave's set-up among them.  At B = 256 that is more than the 16.1 of the kernel that walked rows: what it gains is the order of memory.
#include "fptq_common.h"

namespace fptq {

// 1 / sqrt(2^logb) as the nearest float
constexpr float hadamard_norm(int logb) { return (logb % 2 ? 0x1.6a09e6p-1f : 1.0f) / (float)(1 << (logb / 2)); }

__device__ inline float h_bf16_to_f32(uint32_t bits) { return __uint_as_float(bits << 16); }

// one butterfly stage over registers
template <int S, int V>
__device__ inline void register_stage(float (&v)[V])
{
#pragma unroll
    for (int j = 0; j < V; ++j)
        if ((j & S) == 0) {
            const float a = v[j], b = v[j + S];
            v[j] = a + b;
            v[j + S] = a - b;
        }
}

// One butterfly stage over lanes, an instruction a value: own + sgn * other, with sgn = 1 in a pair's lower lane (a + b) and -1 in its upper
// one, where that is -(a - b): exactly the difference with its sign changed (a product with +-1 and one rounding).  Later stages pair lanes of the same
// sign, so it stays the lane's and goes into the quantizer's multiplier, exactly again.  A DPP operand needs two wait states
// after the instruction that wrote it.
#define FPTQ_LANE_STAGE(name, ctrl)                                                                                                     \
    template <int V>                                                                                                                    \
    __device__ inline void name(float (&v)[V], float sgn)                                                                               \
    {                                                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < V; i += 8) asm("s_nop 1\n\t"                                                              \
            "v_fmac_f32_dpp %0, %0, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %1, %1, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %2, %2, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %3, %3, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %4, %4, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %5, %5, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %6, %6, %8 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                                         \
            "v_fmac_f32_dpp %7, %7, %8 " ctrl " row_mask:0xf bank_mask:0xf"                                                             \
            : "+v"(v[i]), "+v"(v[i + 1]), "+v"(v[i + 2]), "+v"(v[i + 3]), "+v"(v[i + 4]), "+v"(v[i + 5]), "+v"(v[i + 6]), "+v"(v[i + 7]) \
            : "v"(sgn));                                                                                                                \
    }
FPTQ_LANE_STAGE(lanes_xor1, "quad_perm:[1,0,3,2]")
FPTQ_LANE_STAGE(lanes_xor2, "quad_perm:[2,3,0,1]")
FPTQ_LANE_STAGE(lanes_xor7, "row_half_mirror")
FPTQ_LANE_STAGE(lanes_xor8, "row_ror:8")
#undef FPTQ_LANE_STAGE

// bit S of the register index and bit 5 (LANE 32) or 4 (LANE 16) of the lane change places
template <int LANE, int S, int V>
__device__ inline void swap_with_lanes(float (&v)[V])
{
#pragma unroll
    for (int j = 0; j < V; ++j)
        if ((j & S) == 0) {
            const uint32_t a = __float_as_uint(v[j]), b = __float_as_uint(v[j + S]);
            if (LANE == 32) {
                const auto p = __builtin_amdgcn_permlane32_swap(a, b, false, false);
                v[j] = __uint_as_float(p[0]), v[j + S] = __uint_as_float(p[1]);
            } else {
                const auto p = __builtin_amdgcn_permlane16_swap(a, b, false, false);
                v[j] = __uint_as_float(p[0]), v[j + S] = __uint_as_float(p[1]);
            }
        }
}

// A wave takes a span of SPAN values: CH chunks of eight consecutive values a lane (16-byte loads).  Bits 0 .. 2 of an element's place in the
// span are the value in its chunk, bits 3 .. 6 the low four bits of the lane, the rest lane bits 5 and 4 and the chunk's number:
//     B = 256    lanes: block, block; chunks: bit 7            B = 2048   lanes: bits 8, 7; chunks: bits 10, 9
//     B = 512    lanes: bit 7, block; chunks: bit 8            B = 4096   lanes: bits 8, 7; chunks: bits 11, 10, 9
//     B = 1024   lanes: bits 8, 7;    chunks: bit 9
// The chunks' bits come first.  Bits 8 and 7 then change places with chunk bits that are done (permlane swaps).  Bits 6 .. 3 pair lanes that
// differ by 8, 7, 2 and 1, which DPP reaches: with lane bits l3 .. l0 they are l3, l2, l1 ^ l2, l0 ^ l2.  What is left is in the chunk.  A lane
// ends up with whole words of codes, 16 lanes with the 64 bytes of a row in a K tile.
//
// WALK: `parts` waves share a row and walk its spans.  RMS scale: it comes from the whole row, which every wave of it sums.  Given or none: calls of more spans
// than a launch may have waves.  STREAM: inputs that the
// last-level cache cannot hold (on a faster card than the table's 8192 x 28672 123.0 us, 117.6 with; 4096 x 11008 from the cache 20.7 and 23.6).
//
// PAIRS (B = 512, rows of an odd number of blocks; with RMS scale of one, whose sum the wave then has in registers): a wave takes two consecutive blocks
// whatever rows they are of, `parts` is the blocks of a row.  With half a wave idle at the end of every row, short rows were slower than in the kernel that walked
// rows a block at a time (us, that kernel / half idle / now; in brackets inputs from the cache): 65536 x 512 26.8 / 32.9 / 22.1 (23.0 / 30.7 / 19.3), 30000 x
// 1536 33.1 / 32.5 / 27.7 (26.2 / 29.4 / 23.3), 3000 x 512 3.6 / 4.0 / 3.5, 4096 x 4608 15.6 / 13.3 / 12.6; RMS 65536 x 512 38.6 / 43.4 / 23.6.
enum { SPANS, WALK, PAIRS };
template <int MODE, int LOGB, bool STREAM, int FORM>
__global__ __launch_bounds__(256) void quantize_act_hadamard_kernel(const uint16_t *__restrict__ x, const float *__restrict__ row_in,
                                                                    uint8_t *__restrict__ out, float *__restrict__ row_out, uint32_t parts, uint32_t per_parts,
                                                                    int M, float inv_s_a, int64_t K, float eps)
{
    constexpr int R = LOGB <= 10 ? 1 : LOGB - 9, CH = 1 << R, V = 8 * CH, SPAN = 64 * V, B = 1 << LOGB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t t, part;
    divide((blockIdx.x * 4 + wave) * (FORM == PAIRS ? 2 : 1), parts, per_parts, t, part);
    if (t >= (uint32_t)M) return;                        // whole waves leave; nothing below synchronises
    const uint16_t *row = x + (int64_t)t * K;
    const int l5 = lane >> 5, l4 = lane >> 4 & 1;
    const int chunk = (lane & 12) | ((lane & 3) ^ (lane & 4 ? 3 : 0));       // bits 3 .. 6
    const int from = chunk * 8 + (LOGB == 8 ? (l5 * 2 + l4) * 256 : LOGB == 9 ? l4 * 512 + l5 * 128 : l5 * 256 + l4 * 128);
    constexpr int FROM_STEP = LOGB == 8 ? 128 : LOGB == 9 ? 256 : 512;
    // PAIRS: the second block may be the next row's first, or none
    const bool next_row = FORM == PAIRS && part + 1 == parts, second = !next_row || t + 1 < (uint32_t)M;
    const uint32_t own_t = next_row && l4 ? (second ? t + 1 : t) : t, own_block = FORM == PAIRS && l4 ? (next_row ? 0 : part + 1) : part;
    v4u regs[CH];
    auto load = [&](int64_t at) {
        // lanes of blocks past the row's end (PAIRS: the last row's) repeat the span's first one
        const int live = FORM == PAIRS ? (second ? SPAN : B) : (int)min((int64_t)SPAN, K - at);
        const v4u *src = reinterpret_cast<const v4u *>(row + at + (SPAN > B && from >= live ? from % B : from));
#pragma unroll
        for (int r = 0; r < CH; ++r) regs[r] = STREAM ? __builtin_nontemporal_load(src + r * (FROM_STEP / 8)) : src[r * (FROM_STEP / 8)];
    };
    int64_t at = (int64_t)part * (FORM == PAIRS ? B : SPAN);
    load(at);

    float s = 1.0f;
    if (MODE == FPTQ_SCALE_RMS) {                        // S_t from the row as the norm layer sees it
        double ss = 0.0;
        auto add = [&](const uint32_t (&w)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double a = (double)h_bf16_to_f32(w[j] & 0xffffu), b = (double)h_bf16_to_f32(w[j] >> 16);
                ss = __builtin_fma(a, a, ss);
                ss = __builtin_fma(b, b, ss);
            }
        };
        if (FORM == PAIRS) {                                     // rows of one block, which the lanes with the same l4 hold
#pragma unroll
            for (int r = 0; r < CH; ++r) add({regs[r].x, regs[r].y, regs[r].z, regs[r].w});
        } else {
            for (int64_t k0 = (int64_t)lane * 8; k0 < K; k0 += 512) {
                const uint4 u = *reinterpret_cast<const uint4 *>(row + k0);
                add({u.x, u.y, u.z, u.w});
            }
        }
        ss = wave_sum<FORM != PAIRS>(ss);
        s = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    } else if (MODE == FPTQ_SCALE_GIVEN) {
        s = row_in[own_t];
    }
    if (FORM == PAIRS) {
        if ((lane & ~16) == 0 && own_block == 0 && (l4 == 0 || second) && row_out) row_out[own_t] = s;
    } else if (lane == 0 && part == 0 && row_out) {
        row_out[t] = s;
    }
    auto sign = [&](int bit) { return chunk & bit ? -1.0f : 1.0f; };
    const float c = ((MODE == FPTQ_SCALE_NONE) ? inv_s_a : s * inv_s_a) * hadamard_norm(LOGB) * (sign(1) * sign(2) * sign(4) * sign(8));

    const int tile_l = LOGB == 8 ? l5 * 4 + l4 * 2 : LOGB == 9 ? (FORM == PAIRS ? 0 : l4 * 4) + l5 * 2 : LOGB == 10 ? l5 * 4 + l4 * 2 : LOGB == 11 ? l5 * 8 + l4 * 4 : l5 * 16 + l4 * 8;
    for (;;) {
        float v[V], squares = 0.0f;
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const uint32_t w[4] = {regs[r].x, regs[r].y, regs[r].z, regs[r].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[8 * r + 2 * j] = __uint_as_float(w[j] << 16), v[8 * r + 2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
                squares = add_squares(squares, w[j]);
            }
        }
        const bool tame = __builtin_amdgcn_ballot_w64(!(squares < TAME && __builtin_fabsf(c) < TAME)) == 0;
        const int64_t here = at;
        at += (int64_t)parts * SPAN;
        if (FORM == WALK && at < K) load(at);
        if constexpr (R == 3) register_stage<32>(v);
        if constexpr (R >= 2) register_stage<16>(v);
        register_stage<8>(v);
        constexpr int S5 = 8 << (R - 1), S4 = R == 1 ? 8 : S5 / 2;
        if constexpr (LOGB >= 9) swap_with_lanes<32, S5>(v), register_stage<S5>(v);
        if constexpr (LOGB >= 10) swap_with_lanes<16, S4>(v), register_stage<S4>(v);
        lanes_xor8(v, sign(8));
        lanes_xor7(v, sign(4));
        lanes_xor2(v, sign(2));
        lanes_xor1(v, sign(1));
        register_stage<4>(v);
        register_stage<2>(v);
        register_stage<1>(v);
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            uint32_t w;
            if (tame) {
                w = quantize_tame(v + 8 * r, c);
            } else {
                w = CODE_TO_NIBBLES;
#pragma unroll
                for (int e = 0; e < 8; ++e) w ^= quant_code(v[8 * r + e], c, 8) << (4 * e);
            }
            // K tile of the chunk: the bits that the swaps have left in its number, and in lane bits 5 and 4
            const int64_t tile = (FORM == PAIRS ? (int64_t)own_block * (B / KT) : here / KT) + tile_l + (LOGB <= 11 ? r : (r & 1) * 4 + (r >> 2) * 2 + (r >> 1 & 1));
            if (FORM == PAIRS ? l4 == 0 || second : SPAN == B || tile * KT < K) *reinterpret_cast<uint32_t *>(out + (tile * M + own_t) * SEG + chunk * 4) = w;
        }
        if (FORM != WALK || at >= K) return;
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
__device__ inline void butterflies16(float (&v)[16])
{
    register_stage<8>(v);
    register_stage<4>(v);
    register_stage<2>(v);
    register_stage<1>(v);
}

template <int MODE, int LOGB>
__global__ __launch_bounds__(1 << (LOGB - 4)) void quantize_act_hadamard_group_kernel(const uint16_t *__restrict__ x, const float *__restrict__ row_in,
                                                                                     uint8_t *__restrict__ out, float *__restrict__ row_out, uint32_t blocks,
                                                                                     uint32_t per_blocks, int M, float inv_s_a, int64_t K)
{
    static_assert(LOGB == 11 || LOGB == 12, "views of four bits");
    constexpr int B = 1 << LOGB, THREADS = B / 16, LOW = LOGB - 8;      // LOW bits below the second view's four
    __shared__ __attribute__((aligned(16))) float lds[B + B / 4 + (16 << LOW)];
    auto word = [](int e) { return e + 4 * (e >> 4) + ((e >> (LOGB - 4)) << LOW); };
    const int t = threadIdx.x;
    uint32_t m, blk;
    divide(blockIdx.x, blocks, per_blocks, m, blk);
    const uint16_t *row = x + (int64_t)m * K, *src = row + (int64_t)blk * B;
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = h_bf16_to_f32(src[j * THREADS + t]);

    float r = 1.0f;
    if (MODE == FPTQ_SCALE_GIVEN) r = row_in[m];
    const float c = ((MODE == FPTQ_SCALE_NONE) ? inv_s_a : r * inv_s_a) * hadamard_norm(LOGB);
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
    if constexpr (LOGB == 12) register_stage<8>(v);
    register_stage<4>(v);
    register_stage<2>(v);
    register_stage<1>(v);
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
    const uint32_t blocks = (uint32_t)(K >> LOGB);
    const dim3 grid((unsigned)(M * blocks)), block(1 << (LOGB - 4));
    if (mode == FPTQ_SCALE_GIVEN)
        quantize_act_hadamard_group_kernel<FPTQ_SCALE_GIVEN, LOGB><<<grid, block, 0, s>>>(x, row_in, out, row_out, blocks, reciprocal(blocks), (int)M, inv_s_a, K);
    else
        quantize_act_hadamard_group_kernel<FPTQ_SCALE_NONE, LOGB><<<grid, block, 0, s>>>(x, row_in, out, row_out, blocks, reciprocal(blocks), (int)M, inv_s_a, K);
    return hipGetLastError();
}

// The scale given or none: a wave per span.  RMS: every wave of a row sums the whole row again, which only pays while there are few rows (2048 x 28672
// in workgroups per block 64 -> 223 us); up to 256 of them are dealt to as many waves as it takes to have about 4096.
template <int LOGB>
static hipError_t launch_spans(const uint16_t *x, int64_t M, int64_t K, int mode, float eps, const float *row_in, float inv_s_a, uint8_t *out,
                               float *row_out, hipStream_t s)
{
    constexpr int64_t SPAN = LOGB <= 10 ? 1024 : 1 << LOGB;
    if (M > MAX_WAVES) return hipErrorInvalidConfiguration;
    int64_t parts = (K + SPAN - 1) / SPAN, waves = M * parts;
    const bool rms = mode == FPTQ_SCALE_RMS, stream = M * K * 2 > ((int64_t)256 << 20);
    const bool pairs = LOGB == 9 && K % 1024 == 512 && (!rms || K == 512) && M * (K / 512) <= 2 * MAX_WAVES, walk = !pairs && (rms || waves > MAX_WAVES);
    if (pairs) {
        parts = K / 512;
        waves = (M * parts + 1) / 2;
    } else if (walk) {
        const int64_t want = !rms ? MAX_WAVES / M : M > 256 ? 1 : (4096 + M - 1) / M;
        parts = parts < want ? parts : want;
        waves = M * parts;
    }
    const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
#define FPTQ_LAUNCH_SPANS(MODE, STREAM, FORM) \
    quantize_act_hadamard_kernel<MODE, LOGB, STREAM, FORM><<<grid, block, 0, s>>>(x, row_in, out, row_out, (uint32_t)parts, reciprocal((uint32_t)parts), (int)M, inv_s_a, K, eps)
    if constexpr (LOGB == 9) {
        if (pairs) {
            if (rms) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_RMS, false, PAIRS);
            else if (mode == FPTQ_SCALE_GIVEN && stream) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_GIVEN, true, PAIRS);
            else if (mode == FPTQ_SCALE_GIVEN) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_GIVEN, false, PAIRS);
            else if (stream) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_NONE, true, PAIRS);
            else FPTQ_LAUNCH_SPANS(FPTQ_SCALE_NONE, false, PAIRS);
            return hipGetLastError();
        }
    }
    if (rms) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_RMS, false, WALK);                   // reads the row twice
    else if (mode == FPTQ_SCALE_GIVEN && walk) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_GIVEN, true, WALK);
    else if (mode == FPTQ_SCALE_GIVEN && stream) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_GIVEN, true, SPANS);
    else if (mode == FPTQ_SCALE_GIVEN) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_GIVEN, false, SPANS);
    else if (walk) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_NONE, true, WALK);
    else if (stream) FPTQ_LAUNCH_SPANS(FPTQ_SCALE_NONE, true, SPANS);
    else FPTQ_LAUNCH_SPANS(FPTQ_SCALE_NONE, false, SPANS);
#undef FPTQ_LAUNCH_SPANS
    return hipGetLastError();
}

hipError_t launch_quantize_act_hadamard(const uint16_t *x, int64_t M, int64_t K, int hadamard_block, int mode, float eps,
                                        const float *row_in, float inv_s_a, uint8_t *out, float *row_out, hipStream_t s)
{
    // Up to 32768 large blocks: a workgroup per block, which is done sooner with one and keeps more of a row's loads in flight (graph of calls, us, a wave
    // per block behind it; in brackets inputs from the cache: 1 x 14336 2.6, 2.95; 512 x 14336 6.7, 7.4; 4096 x 14336 33.0, 32.9 (27.7, 28.8); 1 x 28672 2.8, 4.3;
    // 1024 x 28672 17.6, 19.7 (16.0, 18.1); 2048 x 28672 34.0, 34.7 (28.5, 31.3); beyond: 8192 x 14336 66, 63)
    const bool few = mode != FPTQ_SCALE_RMS && M <= 32768 && M * (K / hadamard_block) <= 32768;
    if (few && hadamard_block == 2048) return launch_group<11>(x, M, K, mode, row_in, inv_s_a, out, row_out, s);
    if (few && hadamard_block == 4096) return launch_group<12>(x, M, K, mode, row_in, inv_s_a, out, row_out, s);
    switch (hadamard_block) {
    case 256: return launch_spans<8>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 512: return launch_spans<9>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 1024: return launch_spans<10>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 2048: return launch_spans<11>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    case 4096: return launch_spans<12>(x, M, K, mode, eps, row_in, inv_s_a, out, row_out, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fptq
