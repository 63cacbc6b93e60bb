// Large-problem kernel of the quantized linear layer: the INT4 x INT4 product on the 6-bit float matrix cores, which run at
// twice the rate of the 8-bit integer ones, with the same integers as result.
//
// Why it is exact.  The FP6 format e2m3 holds every integer -15 .. 15 in units of 1/8 as sign and magnitude (its subnormals
// and its first normal binade have the same spacing): the activations q in [-8, 7] fit, and so do the weights as w + 8 in
// [0, 15].  Products are multiples of 1/64 and the sums stay below 2^24 of them (|q w| <= 64 per term once the +8 is taken
// out, K <= 131071), so the fp32 accumulator never rounds; measured on the device with accumulators up to 2^24 - 1 and
// products from 1 to 225, positive, negative and mixed.  The accumulators start at -8 sum_k q (every token's own constant), so
// what they hold at the end is sum_k q w and not sum_k q (w + 8).
//
// Data flow.  A small kernel first widens the packed activations to six bits in a scratch buffer of the caller (0.75 bytes a
// value, read and written once: 15 us at 8192 x 8192 beside 1637 us of a 57344-channel product), with their signs resolved, and sums each
// token's codes.  The matrix kernel copies those to LDS with buffer loads that write LDS directly, and reads the weights as
// they are, packed: each of its four waves owns 64 channels and all tokens of the tile (256, 192 or 128), so a weight is loaded by one
// wave only, into registers (256 and 192 tokens) or through LDS of the wave's own (128), and its nibbles are spread to six-bit fields by
// 18 VALU instructions per 32 values, 2.25 per MFMA.  Widening both operands in the kernel would take 5.7 VALU instructions per MFMA, and one wave
// per SIMD issues at most eight instructions in the 32 cycles of an MFMA: measured at the INT8 loop's rate.  Widening the
// weights beforehand as well would cost 1.25 bytes of traffic per weight and call, 5 % at 8192 tokens.
//
// What bounds it: the board's power, and the cycles without an MFMA in flight.  On uniform random INT4 operands 8192 x 57344 x 8192 takes
// 1653 us, widening included (4660 TOP/s; boards differ by 4 %), the INT8 kernel 2537, on all-zero operands 1090.  The matrix pipe is
// busy in 66 % of the cycles at about 1.9 of 2.4 GHz.  An MFMA-only loop on such operands that never change reaches 6700 TOP/s, with
// this kernel's LDS reads of activations 5900 to 6250.
#include <cstdio>
#include <type_traits>

#include "fptq_common.h"

namespace fptq {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v12i __attribute__((ext_vector_type(12)));
typedef float v16f __attribute__((ext_vector_type(16)));

typedef __attribute__((address_space(3))) const uint8_t lds_u8;
typedef __attribute__((address_space(3))) const v4i lds_v4i;

// ---- six-bit activations in the scratch buffer: blocks of (K tile, 32 rows), 3 KB each, row blocks innermost, so that a tile of any
// number of blocks is one run.  A block is six planes [half][piece][row] of 16-byte pieces: half h of a row holds its values 64 h ..
// 64 h + 63 as 48 bytes of six-bit fields, i.e. three pieces.  The matrix kernel copies blocks to LDS as they are, and a wave's fragment
// read (one piece of 32 rows per half) is contiguous: no bank conflicts, no swizzle, and all of it in 16-byte reads (the 24 bytes of one
// operand read as 16 + 8 made LDS the bound: 1627 instead of 1227 us on zero operands at 8192 x 57344 x 8192).
constexpr int X6_ROWS = 32, X6_PLANE = X6_ROWS * 16, X6_BLOCK = 6 * X6_PLANE;
constexpr int X6_PAD = 256;                     // rows are padded to a multiple of this
static int64_t x6_rows(int64_t M) { return (M + X6_PAD - 1) / X6_PAD * X6_PAD; }
static int64_t x6_slab(int64_t M) { return x6_rows(M) * (X6_BLOCK / X6_ROWS); }      // bytes per K tile

// (a & m) ^ t in one instruction
__device__ inline uint32_t masked_xor(uint32_t a, uint32_t m, uint32_t t) { return __builtin_amdgcn_bitop3_b32(a, m, t, 0x6A); }

// The 16 nibbles of two dwords to the low four bits of 16 six-bit fields (96 bits), in an order that needs few instructions
// (both operands use it, so it does not matter which).  A nibble can keep its place in a field that starts at a multiple of 12
// bits from it, and reaches the fields in between by a shift of two; field 5 straddles two dwords, and its upper half comes
// out of the funnel shift that moves the other dword.  FLIP inverts every nibble's top bit: two's complement to value + 8.
template <bool FLIP>
__device__ inline uint32_t spread6_part(uint32_t a, uint32_t b, int part)
{
    const uint32_t a2 = a << 2, b2 = __builtin_amdgcn_alignbit(b, a, 30);      // b2: b << 2, a's top two bits below
    if (part == 0) return masked_xor(a2, 0xC03C03C0u, masked_xor(a, 0x0F00F00Fu, FLIP ? 0x08208208u : 0u));
    if (part == 1) return masked_xor(b2, 0x00000003u, masked_xor(a2, 0x03C03C00u, masked_xor(b, 0xF00F00F0u, FLIP ? 0x82082082u : 0u)));
    return masked_xor(b2, 0x3C03C03Cu, masked_xor(b, 0x00F00F00u, FLIP ? 0x20820820u : 0u));
}
template <bool FLIP>
__device__ inline void spread6(uint32_t a, uint32_t b, uint32_t (&o)[3])
{
#pragma unroll
    for (int p = 0; p < 3; ++p) o[p] = spread6_part<FLIP>(a, b, p);
}

// eight two's complement nibbles as magnitudes and sign bits
__device__ inline void sign_magnitude(uint32_t u, uint32_t &mag, uint32_t &sgn)
{
    sgn = (u >> 3) & 0x11111111u;
    mag = (u ^ ((sgn << 4) - sgn)) + sgn;          // where negative (15 - u) + 1: at most 8, no carry out of a nibble
}

// 32 activations to six-bit sign and magnitude
__device__ inline void widen_signed(v4i p, uint32_t *f)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t ma, sa, mb, sb, m[3], s[3];
        sign_magnitude((uint32_t)p[2 * h], ma, sa);
        sign_magnitude((uint32_t)p[2 * h + 1], mb, sb);
        spread6<false>(ma, mb, m);
        spread6<false>(sa, sb, s);                 // bit 0 of every field; the sign is bit 5: the 96 bits shifted by five
        f[3 * h + 0] = m[0] | (s[0] << 5);
        f[3 * h + 1] = m[1] | __builtin_amdgcn_alignbit(s[1], s[0], 27);
        f[3 * h + 2] = m[2] | __builtin_amdgcn_alignbit(s[2], s[1], 27);
    }
}

// Packed activations -> six-bit blocks, and -sum_k q / 8 of every token (the accumulators' start in units of 1/64 is -8 sum).
// A wave takes 32 rows, half a K tile row per lane; the workgroup's waves and the gridDim.y workgroups of a row group take K
// tiles in turn.  Bound by HBM: 0.5 bytes read and 0.75 written per value.
constexpr int CV_WAVES = 8, CV_ROWS = 32, CV_MAX_SPLIT = 4;

__global__ __launch_bounds__(64 * CV_WAVES) void widen_activations_kernel(const uint8_t *__restrict__ xq, int M, int64_t slab, int ktiles,
                                                                          uint8_t *__restrict__ x6, float *__restrict__ start, int rows)
{
    __shared__ int32_t red[CV_WAVES][CV_ROWS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = blockIdx.x * CV_ROWS + (lane >> 1), h = lane & 1;
    const int src_row = min(row, M - 1);           // rows past the end repeat the last one: their outputs are never stored
    uint8_t *const dst = x6 + (int64_t)(row / X6_ROWS) * X6_BLOCK + 3 * h * X6_PLANE + (row % X6_ROWS) * 16;
    int32_t sum = 0;
    for (int kt = blockIdx.y * CV_WAVES + wave; kt < ktiles; kt += CV_WAVES * gridDim.y) {
        const v4i *src = reinterpret_cast<const v4i *>(xq + ((int64_t)kt * M + src_row) * SEG + h * 32);
        const v4i p0 = src[0], p1 = src[1];
        uint32_t f[12];
        widen_signed(p0, f);
        widen_signed(p1, f + 6);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sum = __builtin_amdgcn_sdot8(p0[e], 0x11111111, sum, false);
            sum = __builtin_amdgcn_sdot8(p1[e], 0x11111111, sum, false);
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
            *reinterpret_cast<v4i *>(dst + kt * slab + j * X6_PLANE) = v4i{(int)f[4 * j], (int)f[4 * j + 1], (int)f[4 * j + 2], (int)f[4 * j + 3]};
    }
    sum += __shfl_xor(sum, 1, 64);
    if (h == 0) red[wave][lane >> 1] = sum;
    __syncthreads();
    if (tid < CV_ROWS) {
        int32_t s = 0;
#pragma unroll
        for (int w = 0; w < CV_WAVES; ++w) s += red[w][tid];
        start[(int64_t)blockIdx.y * rows + blockIdx.x * CV_ROWS + tid] = (float)s * -0.125f;      // one partial per workgroup of the row group
    }
}

// Tile 256 (n) x 32 TM (m), four waves of 64 x 32 TM, 32 TM accumulator registers a lane, one workgroup per CU.  K tile 128.  STAGES K
// tiles of activations in an LDS ring; of packed weights DEPTH K tiles in registers, or (W_LDS) the ring's STAGES.  In operand order a
// load touches 32 rows, a quarter of each row's 64 bytes twice, and every line is touched by two loads: four times the tag lookups of
// a contiguous copy, which by all signs bounds what a CU has in flight.  A large tile's MFMAs cover that; on a small one the latency of HBM showed,
// with three and with six K tiles ahead: 1000 x 5120 x 13824 took 73 us on weights from HBM (53 from the last-level cache), 589 x 7391 x
// 17552 91 (67); copied to LDS as they lie and read back 61 (52) and 77 (62).  Where the CUs are full and the weights are in
// the cache the extra LDS traffic costs up to 4 % (2048 x 4096 x 11008 54 -> 56, from HBM 63 -> 57).  256 tokens (TM = 8) widen each weight
// for eight MFMAs, 128 (TM = 4) for four and load twice the weights per operation; the small tiles are for problems that the large one
// cuts into fewer pieces than there are CUs, or into a few more: weights from HBM, 1000 x 5120 x 13824 takes 60 us with 128 tokens, 67 with
// 192, 88 with 256 and 70 on INT8 tiles, 333 x 32000 x 4096 50, 36, 40 and 46.
//
// DEPTH 3 takes a loop unrolled by six (W sets in twos, packed sets in threes), DEPTH 2 by two.  A launch of few K tiles goes through most of the code of six
// once or twice, at the speed at which code arrives, on some cards slower than the MFMAs; so up to 32 K tiles take DEPTH 2.  us, weights from HBM, DEPTH 3 / 2, on a
// card where code arrives slowly and on one where it arrives fast: 333 x 32000 x 2504 28.0 / 26.7, 25.8 / 25.1; 333 x 32003 x 2504 with its quantizer 30.8 / 29.8,
// 29.4 / 29.4; 2048 x 22016 x 1280 49.2 / 48.3, 45.4 / 44.8; 333 x 32000 x 4096 33.1 / 32.8, 32.5 / 32.6.  From there on two K tiles ahead count for more: 500 x 21000
// x 8192 54.8 / 56.8, 1500 x 14336 x 6144 74.4 / 75.5.  128 tokens keep six at any length (W_LDS; unrolled by two 1000 x 5120 x 2504 15.6 -> 16.0).
template <int TM_, int DEPTH_>
struct PrefillTile {
    static constexpr int TN = 2, TM = TM_, STAGES = 5, DEPTH = DEPTH_, UNROLL = DEPTH == 2 ? 2 : 6;
    static constexpr bool W_LDS = TM == 4;          // five stages of both operands are 140 of the 160 KB of LDS; a larger tile's would not fit
    static constexpr int BN = 4 * TN * 32, BM = TM * 32;
    static constexpr int X_BYTES = BM * (X6_BLOCK / X6_ROWS), W_BYTES = TN * 32 * SEG;          // 3 KB per 32 tokens; a wave's 4 KB of weights
    // vector loads of a wave per K tile: equally many for each wave, so that the waves can count them; the last ones may have nothing to copy
    static constexpr int FILLS = (X_BYTES + 4095) / 4096, W_LOADS = 2 * TN, LOADS = FILLS + W_LOADS;
    static constexpr int X_LDS = FILLS * 4096, STAGE_BYTES = X_LDS + (W_LDS ? 4 * W_BYTES : 0);
    // the loop issues the weights' loads in groups 0 and 1 of its TM groups of MFMAs, two fills in group 2, and one in each after that
    static constexpr int BEFORE_LAST = W_LOADS + 2;                                             // loads issued before the last group (W_LDS: four groups)
    static constexpr int RING_BYTES = STAGES * STAGE_BYTES, LDS_BYTES = RING_BYTES + (2 * BN + BM) * 4;
    static_assert(TM >= 4 && TM <= 8 && 2 + TM - 3 >= FILLS, "a group for every load");
    static_assert(LDS_BYTES <= 160 * 1024, "");
    static_assert(W_LDS || (DEPTH >= STAGES - 3 && DEPTH <= STAGES - 1), "the wait counts assume weights and fills issued in the loop's order from the start");
};

// 32 x 32 x 64, both operands e2m3 (format code 2): 24 bytes, i.e. the first six registers, of each operand are read
__device__ inline v16f mfma6(v8i w, v8i x, v16f c)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, x, c, 2, 2, 0, 0, 0, 0);
}

template <int TM, int STORE, bool DUMP, bool ZP, int DEPTH>
__global__ __launch_bounds__(256, 1) void linear_prefill_kernel(
    const uint8_t *__restrict__ x6, int64_t x_slab, const float *__restrict__ start, int start_parts, int rows,
    const uint8_t *__restrict__ wq, int M, int N, int ktiles, int tiles_m, int tiles_n, float s_a, const float *__restrict__ s_w,
    const float *__restrict__ d, int zp, const int32_t *__restrict__ wsum, uint16_t *__restrict__ y, int32_t *__restrict__ acc_out)
{
    typedef PrefillTile<TM, DEPTH> C;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = lane & 31, fg = lane >> 5;

    // ---- tile of this workgroup: a contiguous run of tiles per XCD (workgroups are dealt to the 8 XCDs in turn), in bands of 8
    // N-tiles with M fastest, so that the tiles an XCD runs together share panels in its L2
    const int total = tiles_m * tiles_n;
    int pid = blockIdx.x;
    {
        const int per = (total + 7) / 8, tall = total % 8 == 0 ? 8 : total % 8;
        const int xcd = pid % 8, local = pid / 8;
        pid = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
    }
    constexpr int GN = 8;
    const int band = pid / (GN * tiles_m), in_band = pid % (GN * tiles_m);
    const int band_w = min(GN, tiles_n - band * GN);
    const int bn = band * GN + in_band % band_w, bm = in_band / band_w;
    const int m0 = bm * C::BM, nw0 = bn * C::BN + wave * (C::TN * 32);

    // ---- activations, HBM -> LDS: one run of 3 TM KB per K tile, a quarter of it per wave.  Past the last K tile the descriptor is
    // empty: the loads are still issued (the wait counts stay the same) and land as zeros.
    const int x_voff = bm * C::X_BYTES + wave * (C::FILLS * 1024) + lane * 16;
    const int x_end = min((int)x_slab, (bm + 1) * C::X_BYTES);      // past it lie other tiles' rows, or none
    uint8_t *const fill_base = lds + wave * (C::FILLS * 1024);
    auto fill1 = [&](auto jc, __amdgpu_buffer_rsrc_t r, uint8_t *to) {
        constexpr int J = decltype(jc)::value;     // 1 KB; the instruction's offset moves both addresses
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, LDS_PTR(to + J / 3 * 3072), 16, x_voff + J / 3 * 3072, 0, J % 3 * 1024, 0);
    };
    auto fill_from = [&](auto from, auto n, __amdgpu_buffer_rsrc_t r, uint8_t *to) {       // n of the loads of a K tile
        constexpr int J = decltype(from)::value, N_ = decltype(n)::value;
        if constexpr (N_ > 0) fill1(std::integral_constant<int, J>(), r, to);
        if constexpr (N_ > 1) fill1(std::integral_constant<int, J + 1>(), r, to);
        if constexpr (N_ > 2) fill1(std::integral_constant<int, J + 2>(), r, to);
        if constexpr (N_ > 3) fill1(std::integral_constant<int, J + 3>(), r, to);
        if constexpr (N_ > 4) fill1(std::integral_constant<int, J + 4>(), r, to);
        if constexpr (N_ > 5) fill1(std::integral_constant<int, J + 5>(), r, to);
    };
    auto slab_desc = [&](const uint8_t *p, int64_t bytes, bool in) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, in ? (int)bytes : 0, RSRC_FLAGS);
    };
    // ---- weights, HBM -> registers (W_LDS: LDS -> registers): lane (fi, fg) loads half fg (granules 2 fg, 2 fg + 1) of row nw0 + 32 t + fi, the k values of
    // the activations' half fg; rows past N read as zero
    const int64_t w_slab = (int64_t)N * SEG;
    const int w_voff = (nw0 + fi) * SEG + fg * 32;
    constexpr int RAWS = C::W_LDS ? 2 : C::DEPTH;          // sets of packed weights: being widened and being read, or in flight
    v4i raw[RAWS][2][C::TN];
    auto load_w1 = [&](__amdgpu_buffer_rsrc_t r, int s, int t) {
        return __builtin_amdgcn_raw_buffer_load_b128(r, w_voff + t * (32 * SEG) + s * 16, 0, 0);
    };
    // W_LDS: a wave first copies the 4 KB of its rows as they lie in HBM to its own part of the ring's stage, behind the activations, the
    // 16-byte granules of a row permuted (granule g of row r in slot g ^ (r / 4) % 4) so that the reads back are free of bank conflicts.
    const int w_lane = (nw0 + (lane >> 2)) * SEG + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
    uint8_t *const w_fill_base = lds + C::X_LDS + wave * C::W_BYTES;
    auto w_fill1 = [&](auto jc, __amdgpu_buffer_rsrc_t r, uint8_t *to) {
        constexpr int J = decltype(jc)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, LDS_PTR(to), 16, w_lane, 0, J * 1024, 0);
    };
    lds_u8 *const w_base = (lds_u8 *)lds + C::X_LDS + wave * C::W_BYTES + fi * SEG;
    const int w_slot0 = ((2 * fg) ^ ((fi >> 2) & 3)) << 4;
    auto read_w1 = [&](int stage_off, v4i (&r)[2][C::TN], int i) { r[i % 2][i / 2] = *(lds_v4i *)(w_base + stage_off + i / 2 * (32 * SEG) + (w_slot0 ^ (i % 2 * 16))); };
    auto read_w = [&](int stage_off, v4i (&r)[2][C::TN]) { read_w1(stage_off, r, 0), read_w1(stage_off, r, 1), read_w1(stage_off, r, 2), read_w1(stage_off, r, 3); };
    // ---- fragments: the 48 bytes of token 32 x + fi, half fg; the first 24 feed MFMA step 0, the others step 1
    lds_u8 *const x_base = (lds_u8 *)lds + fg * (3 * X6_PLANE) + fi * 16;
    v12i X[C::TM];
    auto read_piece = [&](int stage_off, int x, int p) {       // 16 of the 48 bytes
        const v4i a = *(lds_v4i *)(x_base + stage_off + x * X6_BLOCK + p * X6_PLANE);
#pragma unroll
        for (int e = 0; e < 4; ++e) X[x][4 * p + e] = a[e];
    };
    auto read_x = [&](int stage_off, int x) { read_piece(stage_off, x, 0), read_piece(stage_off, x, 1), read_piece(stage_off, x, 2); };

    // ---- the accumulators' start: partial sums of the widening kernel's workgroups, all fetched at once (missing ones read as
    // zero) and ahead of everything else, so that they cost no round trip of their own
    const __amdgpu_buffer_rsrc_t sr = slab_desc(reinterpret_cast<const uint8_t *>(start), (int64_t)start_parts * rows * 4, true);
    // Both halves of a wave need the same tokens' sums, so each fetches half of the parts (a load occupies the address unit whatever it fetches).
    static_assert(CV_MAX_SPLIT == 4, "two parts for each half of the wave");
    float sv[C::TM][2];
#pragma unroll
    for (int x = 0; x < C::TM; ++x)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            sv[x][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, ((2 * fg + i) * rows + m0 + x * 32 + fi) * 4, 0, 0));

    // ---- what the epilogue multiplies by: a channel per thread (its wave's own), a token per thread.  Fetched here and kept in LDS
    // behind the ring: the epilogue would wait for the channels' once per tile and for the tokens' once per 32 of them (4096 x 28672 x
    // 4096 266 us against 261, with token scales 271 against 260).
    float *const cwbuf = reinterpret_cast<float *>(lds + C::RING_BYTES), *const zwbuf = cwbuf + C::BN, *const dbuf = zwbuf + C::BN;
    const int cn = min(bn * C::BN + tid, N - 1);
    const float cw0 = s_w[cn], zw0 = ZP ? (float)(zp * wsum[cn]) : 0.0f;
    const float d0 = d && tid < C::BM ? d[min(m0 + tid, M - 1)] : 1.0f;

    // ---- prologue: the loop's loads in the loop's order (iteration j issues the weights of tile j + DEPTH, with W_LDS of tile
    // j + STAGES - 1, then the fill of tile j + STAGES - 1), from an empty pipeline
    const uint8_t *wp = wq, *xp = x6;              // next tile to load; they run past the end with empty descriptors
    int w_left = ktiles, x_left = ktiles;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 1 - C::STAGES; j < 0; ++j) {
        if constexpr (C::W_LDS) {
            const __amdgpu_buffer_rsrc_t r = slab_desc(wp, w_slab, w_left-- > 0);
            wp += w_slab;
            uint8_t *const to = w_fill_base + (j + C::STAGES - 1) * C::STAGE_BYTES;
            w_fill1(std::integral_constant<int, 0>(), r, to), w_fill1(std::integral_constant<int, 1>(), r, to);
            w_fill1(std::integral_constant<int, 2>(), r, to), w_fill1(std::integral_constant<int, 3>(), r, to);
        } else if (j + C::DEPTH >= 0) {
            const __amdgpu_buffer_rsrc_t r = slab_desc(wp, w_slab, w_left-- > 0);
            wp += w_slab;
            v4i(&rl)[2][C::TN] = raw[j + C::DEPTH < 0 ? 0 : j + C::DEPTH];
#pragma unroll
            for (int t = 0; t < C::TN; ++t) rl[0][t] = load_w1(r, 0, t), rl[1][t] = load_w1(r, 1, t);
        }
        const __amdgpu_buffer_rsrc_t r = slab_desc(xp, x_end, x_left-- > 0);
        xp += x_slab;
        uint8_t *const to = fill_base + (j + C::STAGES - 1) * C::STAGE_BYTES;
        fill_from(std::integral_constant<int, 0>(), std::integral_constant<int, C::FILLS>(), r, to);
        __builtin_amdgcn_sched_barrier(0);
    }
    v16f acc[C::TN][C::TM];
#pragma unroll
    for (int x = 0; x < C::TM; ++x) {
        const uint32_t own = __float_as_uint(sv[x][0] + sv[x][1]);
        const auto both = __builtin_amdgcn_permlane32_swap(own, own, false, false);
        const float v = __uint_as_float(both[0]) + __uint_as_float(both[1]);      // integers: exact in any order
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][x][r] = v;
    }
    cwbuf[tid] = s_a * cw0;
    if (ZP) zwbuf[tid] = zw0;
    if (tid < C::BM) dbuf[tid] = d0;
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
    // weights in registers: at least that many fills are younger than tile 0's; through LDS: tile 1's weights are in as well
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::W_LDS ? C::LOADS * (C::STAGES - 3) : C::FILLS * (C::STAGES - 2)));
    __builtin_amdgcn_s_barrier();
    v8i W[2][2][C::TN];                            // widened weights of this K tile and of the next one: [tile][step][t]
    // A lane widens 128 values per K tile, 16 at a time (h: step h / 4, t = h / 2 % 2), one of the three dwords of fields at a time.
    auto widen_third = [&](const v4i (&r)[2][C::TN], v8i (&w)[2][C::TN], int h, int part) {
        const int s = h / 4, t = (h / 2) % 2, o = h % 2;
        w[s][t][3 * o + part] = (int)spread6_part<true>((uint32_t)r[s][t][2 * o], (uint32_t)r[s][t][2 * o + 1], part);
    };
#pragma unroll
    for (int x = 0; x < C::TM - 1; ++x) read_x(0, x);
    if constexpr (C::W_LDS) read_w(0, raw[0]), read_w(C::STAGE_BYTES, raw[1]);
#pragma unroll
    for (int i = 0; i < 24; ++i) widen_third(raw[0], W[0], i / 3, i % 3);
    __builtin_amdgcn_sched_barrier(0);

    // ---- K loop.  A K tile is TM groups of four MFMAs, group x on the tokens 32 x ..: two steps of 64 values times two runs of 32
    // channels.  Behind every MFMA goes what one wave can issue while it runs, fenced, because the compiler keeps to the order of the source where registers
    // are scarce: a fragment read (three a group: X[x - 1] of the next K tile, in group 0 the last X of this one, whose old value the
    // previous tile's last group still used), a share of the next K tile's weights being widened (9 VALU per 16 values), a load of a later tile.  Four MFMAs
    // followed by all of that, as most groups of the large tiles were, took 1255 clocks a K tile of 256 tokens and 1056 of 192 (1024 and 768 of MFMAs), now
    // 1236 and 957; the clock gives most of it back (1.52 instead of 1.64 GHz at 192 tokens).  The loads of a run of rows go in pairs, so that two loads
    // that touch the same lines (and a wave's copies of one page) meet: 500 x 21000 x 8192 55.1 us apart, 53.5 in pairs, 589 x 7391 x 17552 76.8 and 75.5; all
    // four at once, or all fills at once, is 1 to 5 % slower again.  Together 8192 x 57344 x 8192 1627 -> 1606, 8192 x 8192 x 28672 799 -> 788, 500 x 21000 x
    // 8192 55.4 -> 53.5, 2048 x 4096 x 11008 56.0 -> 55.6.
    int off = 0, off_next = C::STAGE_BYTES, off_prev = C::RING_BYTES - C::STAGE_BYTES;      // ring positions of tiles kt, kt + 1, kt - 1, in bytes
    __amdgpu_buffer_rsrc_t wr = slab_desc(wp, w_slab, w_left > 0), xr = slab_desc(xp, x_end, x_left > 0);
    __builtin_amdgcn_s_setprio(2);
    auto tile = [&](auto pc) {
        constexpr int P = decltype(pc)::value;     // position in the unrolled loop: P % 2 names the W set, P % DEPTH the raw set
        v4i(&load_to)[2][C::TN] = raw[P % RAWS];           // tile kt's, widened during the previous tile
        const v4i(&next)[2][C::TN] = raw[(P + 1) % RAWS];
        uint8_t *const fill_to = fill_base + off_prev, *const w_fill_to = w_fill_base + off_prev;
#pragma unroll
        for (int x = 0; x < C::TM; ++x) {
            asm("" : "+v"(X[x]));           // keeps the 48 bytes in one run of registers, of which both steps' operands are parts
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = i / 2, t = i % 2;
                const v8i b = s == 0 ? __builtin_shufflevector(X[x], X[x], 0, 1, 2, 3, 4, 5, -1, -1)
                                     : __builtin_shufflevector(X[x], X[x], 6, 7, 8, 9, 10, 11, -1, -1);
                acc[t][x] = mfma6(W[P % 2][s][t], b, acc[t][x]);
                __builtin_amdgcn_sched_barrier(0);
                // Before the first read of tile kt + 1: this wave's part of it has landed (younger: whole iterations of loads and this one's of group 0);
                // the barrier extends that to every wave's part, and says every wave has read all of tile kt - 1, whose place the fills
                // from group 2 on take (a wave's own weights in LDS were read before that).
                if (x == (C::W_LDS ? 0 : 1) && i == 0) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::LOADS * (C::STAGES - 3) + (C::W_LDS ? 0 : 2)));
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
                // this wave's weights of tile kt + 2 are in (its own copies: no barrier); younger: an iteration's loads and this one's so far
                if (C::W_LDS && x == C::TM - 1 && i == 0) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::LOADS * (C::STAGES - 4) + C::BEFORE_LAST));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (i < 3) read_piece(x == 0 ? off : off_next, x == 0 ? C::TM - 1 : x - 1, i);
                if (C::W_LDS && x == C::TM - 1) read_w1(off_next + C::STAGE_BYTES == C::RING_BYTES ? 0 : off_next + C::STAGE_BYTES, load_to, i);
                const int slot = 4 * x + i;        // of 4 TM: 24 thirds go into them
#pragma unroll
                for (int k = slot * 6 / C::TM; k < (slot + 1) * 6 / C::TM; ++k) widen_third(next, W[(P + 1) % 2], k / 3, k % 3);
                if constexpr (C::W_LDS) {
                    if (x == 0 && i == 3) w_fill1(std::integral_constant<int, 0>(), wr, w_fill_to), w_fill1(std::integral_constant<int, 1>(), wr, w_fill_to);
                    if (x == 1 && i == 3) w_fill1(std::integral_constant<int, 2>(), wr, w_fill_to), w_fill1(std::integral_constant<int, 3>(), wr, w_fill_to);
                } else {
                    if (x < 2 && i == 3) load_to[0][x] = load_w1(wr, 0, x), load_to[1][x] = load_w1(wr, 1, x);
                }
                if (x == 2 && i == 3) fill_from(std::integral_constant<int, 0>(), std::integral_constant<int, 2>(), xr, fill_to);
                constexpr int REST = C::FILLS - 2;
                if constexpr (REST > 0) { if (x == 3 && i == 1) fill1(std::integral_constant<int, 2>(), xr, fill_to); }
                if constexpr (REST > 1) { if (x == 4 && i == 1) fill1(std::integral_constant<int, 3>(), xr, fill_to); }
                if constexpr (REST > 2) { if (x == 5 && i == 1) fill1(std::integral_constant<int, 4>(), xr, fill_to); }
                if constexpr (REST > 3) { if (x == 6 && i == 1) fill1(std::integral_constant<int, 5>(), xr, fill_to); }
                if (x == C::TM - 1 && i == 3) {    // addresses of the next iteration
                    wp += w_slab, xp += x_slab;
                    --w_left, --x_left;
                    wr = slab_desc(wp, w_slab, w_left > 0), xr = slab_desc(xp, x_end, x_left > 0);
                    off_prev = off, off = off_next, off_next = off_next + C::STAGE_BYTES == C::RING_BYTES ? 0 : off_next + C::STAGE_BYTES;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // unrolled, so that the weights' two or three register sets rotate without copies
    int left = ktiles;
#define FPTQ_TILE(i) tile(std::integral_constant<int, i>())
    if constexpr (C::UNROLL == 2) {
        for (; left >= 2; left -= 2) FPTQ_TILE(0), FPTQ_TILE(1);
        if (left > 0) FPTQ_TILE(0);
    } else {
        for (; left >= 6; left -= 6) FPTQ_TILE(0), FPTQ_TILE(1), FPTQ_TILE(2), FPTQ_TILE(3), FPTQ_TILE(4), FPTQ_TILE(5);
        if (left > 0) FPTQ_TILE(0);
        if (left > 1) FPTQ_TILE(1);
        if (left > 2) FPTQ_TILE(2);
        if (left > 3) FPTQ_TILE(3);
        if (left > 4) FPTQ_TILE(4);
    }
#undef FPTQ_TILE
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the tail loads before LDS is reused
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
    __builtin_amdgcn_s_barrier();

    // ---- epilogue.  Weights were the A operand: a lane owns token fi of each 32 and, per register quad q, four consecutive
    // channels 8 q + 4 fg + (r % 4).  The registers hold acc / 64; times 64 that is acc, exactly, and then
    // y = bf16((float)(acc - z * wsum[n]) * (s_a * s_w[n]) [* d_t]) as in the other kernels (with a zero point the subtraction is
    // exact too: both terms are integers and their difference is below 2^24 for K <= 131071).  Without a zero point the 64 goes into the
    // channel's factor, a power of two and so exact, unless that would overflow it (`huge`, never with real scales).
    //
    // One wave per SIMD has nothing to hide a latency under, so the 32 (64 with a zero point) channel constants are read once, into the
    // registers that the K loop's operands leave free, and the results of a group of 32 tokens are read back from LDS while the next
    // group's are computed and written: 6.1 us a tile with the constants read where they are used and one patch for all groups,
    // 3.6 now (2.8 to 4.2 from workgroup to workgroup).  With token scales and no zero point the registers do not suffice on the 256-token tile: 17
    // go through scratch, 15 operations a lane (2048 x 22016 x 4096 104.9 us, 101.5 without token scales, 102.0 with both).  The two halves of a wave exchange quads, so that a lane holds eight consecutive channels (16 bytes); those go
    // through a wave-private LDS patch of 32 rows of 128 bytes per group, granule g of row r in slot g ^ (r % 8) (no bank
    // conflicts in either direction), so that HBM sees rows of 128 bytes.  A wave's LDS operations complete in order, so only the
    // compiler has to be kept from exchanging them.
    constexpr int WN = C::TN * 32, ROW_BYTES = WN * 2, PATCH_BYTES = 32 * ROW_BYTES;
    static_assert(WN == 64 && 4 * 2 * PATCH_BYTES <= C::RING_BYTES, "a channel per lane; two patches a wave reuse the ring");
    uint8_t *const patch = lds + wave * (2 * PATCH_BYTES);
    float4 cw[C::TN][4], zw[C::TN][4];
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cw[tn][q] = *reinterpret_cast<const float4 *>(cwbuf + wave * WN + tn * 32 + 8 * q + 4 * fg);
            if (ZP) zw[tn][q] = *reinterpret_cast<const float4 *>(zwbuf + wave * WN + tn * 32 + 8 * q + 4 * fg);
        }
    float dm[C::TM];
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) dm[tm] = d ? dbuf[tm * 32 + fi] : 1.0f;
    bool huge = false;
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            huge |= fmaxf(fmaxf(fabsf(cw[tn][q].x), fabsf(cw[tn][q].y)), fmaxf(fabsf(cw[tn][q].z), fabsf(cw[tn][q].w))) >= 0x1p121f;
    const bool plain = !ZP && !d && __builtin_amdgcn_ballot_w64(huge) == 0;
    const int slot = fg ^ (fi & 7);
    // PLAIN: neither zero point nor token scale, and the 64 in the channel's factor
    auto to_lds = [&](auto plain_c, int tm) {
        constexpr bool PLAIN = decltype(plain_c)::value;
        uint8_t *const to = patch + (tm & 1) * PATCH_BYTES + fi * ROW_BYTES;
#pragma unroll
        for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint32_t p[2][2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4 c4 = cw[tn][2 * j + q], z4 = zw[tn][2 * j + q];
                    const float c[4] = {c4.x, c4.y, c4.z, c4.w}, z[4] = {z4.x, z4.y, z4.z, z4.w};
                    float yf[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float a = acc[tn][tm][8 * j + 4 * q + e];
                        yf[e] = PLAIN ? a * c[e] : (ZP ? __builtin_fmaf(a, 64.0f, -z[e]) : a * 64.0f) * c[e] * dm[tm];
                    }
                    p[q][0] = pack_bf16(yf[0], yf[1]), p[q][1] = pack_bf16(yf[2], yf[3]);
                }
                // lanes 32 .. 63 of the first and 0 .. 31 of the second change places: quads 2 j of both halves, and 2 j + 1
                const auto lo = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
                *reinterpret_cast<uint4 *>(to + ((tn * 4 + 2 * j) ^ slot) * 16) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // a store instruction takes eight rows
    const int col = (lane & 7) * 8, row = lane >> 3;
    const uint8_t *const from = patch + row * ROW_BYTES + (((lane & 7) ^ row) << 4);
    const uint32_t y_off = nw0 + col + (STORE == ANY_ALIGNMENT ? 7 : 0) < N ? (uint32_t)row * ((uint32_t)N * 2) + (uint32_t)(nw0 + col) * 2 : 0x80000000u;
    auto write_out = [&](auto plain_c) {
        to_lds(plain_c, 0);
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm) {
            uint4 v[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) v[p] = *reinterpret_cast<const uint4 *>(from + (tm & 1) * PATCH_BYTES + p * (8 * ROW_BYTES));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (tm + 1 < C::TM) to_lds(plain_c, tm + 1);
            store_rows<STORE, 4, 8>(v, y, y_off, m0 + tm * 32, row, nw0 + col, nw0 + col < N, M, N, nw0 + WN > N);
        }
    };
    if (plain) {
#pragma unroll
        for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q) cw[tn][q].x *= 64.0f, cw[tn][q].y *= 64.0f, cw[tn][q].z *= 64.0f, cw[tn][q].w *= 64.0f;
        write_out(std::true_type());
    } else {
        write_out(std::false_type());
    }
    if (DUMP) {      // parity dump of the integer accumulators (never a timed path)
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = m0 + tm * 32 + fi, n = nw0 + tn * 32 + 8 * (r / 4) + 4 * fg + r % 4;
                    if (m < M && n < N) acc_out[(int64_t)m * N + n] = (int32_t)(acc[tn][tm][r] * 64.0f);
                }
    }
}

template <int TM, int STORE, bool DUMP, bool ZP, int DEPTH>
static hipError_t set_prefill_attribute()
{
    return hipFuncSetAttribute((const void *)linear_prefill_kernel<TM, STORE, DUMP, ZP, DEPTH>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               PrefillTile<TM, DEPTH>::LDS_BYTES);
}

template <int TM, int DEPTH>
static hipError_t set_prefill_attributes()
{
    hipError_t e = hipSuccess;
    auto one = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    one(set_prefill_attribute<TM, ANY_ALIGNMENT, true, false, DEPTH>()), one(set_prefill_attribute<TM, ANY_ALIGNMENT, true, true, DEPTH>());
    one(set_prefill_attribute<TM, ANY_ALIGNMENT, false, false, DEPTH>()), one(set_prefill_attribute<TM, ANY_ALIGNMENT, false, true, DEPTH>());
    one(set_prefill_attribute<TM, CACHED, false, false, DEPTH>()), one(set_prefill_attribute<TM, CACHED, false, true, DEPTH>());
    one(set_prefill_attribute<TM, STREAMED, false, false, DEPTH>()), one(set_prefill_attribute<TM, STREAMED, false, true, DEPTH>());
    return e;
}

hipError_t prefill_device_init()
{
    hipError_t e = set_prefill_attributes<8, 3>();
    if (e == hipSuccess) e = set_prefill_attributes<8, 2>();
    if (e == hipSuccess) e = set_prefill_attributes<6, 3>();
    if (e == hipSuccess) e = set_prefill_attributes<6, 2>();
    if (e == hipSuccess) e = set_prefill_attributes<4, 3>();
    return e;
}

// Workgroups per group of 32 rows in the widening kernel: about two per CU in all, each with a K tile per wave at least.
static int widen_split(int64_t M, int64_t K, int cus)
{
    const int64_t groups = x6_rows(M) / CV_ROWS;
    int64_t split = 2 * cus / groups;
    if (split > k_tiles(K) / CV_WAVES) split = k_tiles(K) / CV_WAVES;
    if (split > CV_MAX_SPLIT) split = CV_MAX_SPLIT;
    return split < 1 ? 1 : (int)split;
}

// Scratch: the partial starts [CV_MAX_SPLIT][rows], then the six-bit activations.
static int64_t start_bytes(int64_t M) { return (int64_t)CV_MAX_SPLIT * x6_rows(M) * 4; }
int64_t prefill_scratch_bytes(int64_t M, int64_t K) { return start_bytes(M) + k_tiles(K) * x6_slab(M); }

int64_t prefill_workgroups(int64_t M, int64_t N, int tile_tokens)
{
    return ((M + tile_tokens - 1) / tile_tokens) * ((N + PrefillTile<8, 3>::BN - 1) / PrefillTile<8, 3>::BN);
}

template <int TM, int DEPTH>
static hipError_t launch_tile(const uint8_t *x6, const float *start, int split, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                              const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc, hipStream_t s)
{
    typedef PrefillTile<TM, DEPTH> C;
    const int64_t tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    if (tiles_m * tiles_n > 0x7fffffff) return hipErrorInvalidValue;
#define FPTQ_PREFILL(A, D, Z)                                                                                                        \
    linear_prefill_kernel<TM, A, D, Z, DEPTH><<<dim3((unsigned)(tiles_m * tiles_n)), dim3(256), C::LDS_BYTES, s>>>(                          \
        x6, x6_slab(M), start, split, (int)x6_rows(M), wq, (int)M, (int)N, (int)k_tiles(K), (int)tiles_m, (int)tiles_n, s_a, s_w, d,   \
        zp, wsum, y, acc)
    const bool z = wsum != nullptr;
    if (acc) {
        if (z) FPTQ_PREFILL(ANY_ALIGNMENT, true, true);
        else FPTQ_PREFILL(ANY_ALIGNMENT, true, false);
        return hipGetLastError();
    }
    switch (store_kind(M, N)) {
    case CACHED: if (z) FPTQ_PREFILL(CACHED, false, true); else FPTQ_PREFILL(CACHED, false, false); break;
    case STREAMED: if (z) FPTQ_PREFILL(STREAMED, false, true); else FPTQ_PREFILL(STREAMED, false, false); break;
    default: if (z) FPTQ_PREFILL(ANY_ALIGNMENT, false, true); else FPTQ_PREFILL(ANY_ALIGNMENT, false, false);
    }
#undef FPTQ_PREFILL
    return hipGetLastError();
}

hipError_t launch_linear_prefill(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a, const float *s_w,
                                 const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc, uint8_t *scratch, int tile_tokens,
                                 hipStream_t s)
{
    const DeviceInfo *info;
    hipError_t e = device_info(&info);
    if (e != hipSuccess) return e;
    const int rows = (int)x6_rows(M), split = widen_split(M, K, info->cus);
    float *start = reinterpret_cast<float *>(scratch);
    uint8_t *x6 = scratch + start_bytes(M);
    widen_activations_kernel<<<dim3((unsigned)(rows / CV_ROWS), (unsigned)split), dim3(64 * CV_WAVES), 0, s>>>(
        xq, (int)M, x6_slab(M), (int)k_tiles(K), x6, start, rows);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const bool few = k_tiles(K) <= 32;
#define FPTQ_TOKENS(TM, DEPTH) launch_tile<TM, DEPTH>(x6, start, split, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s)
    switch (tile_tokens) {
    case 128: return FPTQ_TOKENS(4, 3);
    case 192: return few ? FPTQ_TOKENS(6, 2) : FPTQ_TOKENS(6, 3);
    default: return few ? FPTQ_TOKENS(8, 2) : FPTQ_TOKENS(8, 3);
    }
#undef FPTQ_TOKENS
}

}  // namespace fptq
