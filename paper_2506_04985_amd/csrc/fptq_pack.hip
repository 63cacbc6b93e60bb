// Offline packing of INT4 weights into the library layout (two values per byte, App. J of the
// paper), the inverse used by parity checks, and the simple one-thread-per-output linear kernel.
#include "fptq_common.h"

namespace fptq {

// Sixteen int8 values of a row from k0 on, zeros past its end: one 16-byte load at any alignment (the hardware takes it) but at the
// row's ragged end.
__device__ inline uint4 load_row16(const int8_t *__restrict__ row, int64_t k0, int64_t K)
{
    uint4 v = make_uint4(0, 0, 0, 0);
    if (k0 + 16 <= K) {
        __builtin_memcpy(&v, row + k0, 16);
    } else if (k0 < K) {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 15; ++i)
            if (k0 + i < K) w[i >> 2] |= (uint32_t)(uint8_t)row[k0 + i] << (8 * (i & 3));
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return v;
}

// low nibbles of eight bytes -> one word, the first byte's lowest
__device__ inline uint32_t pack8(uint32_t lo, uint32_t hi)
{
    lo &= 0x0F0F0F0Fu, hi &= 0x0F0F0F0Fu;
    lo |= lo >> 4, hi |= hi >> 4;                  // bytes 0 and 2 hold a pair each
    return __builtin_amdgcn_perm(hi, lo, 0x06040200u);
}

// Bound by HBM: a byte read and half a byte written per value.  A thread makes the 16-byte granules (32 values) at one place of
// PACK_TILES K tiles in a row: a wave reads PACK_TILES x 128 contiguous bytes of 16 rows and writes 1 KB runs.  A byte per load, one granule
// per thread, took 221 us at 28672 x 4096; half granules (8 lanes a row) and eight tiles per thread: the same as now.
// ALONG_K: consecutive workgroups take the K tiles of the same rows, so that whole rows are read in one go, otherwise the same K tiles of the next
// rows, which writes longer runs.  The first pays for large matrices whose rows are 4, 8, 12 or 16 KB (integers from HBM, across / along K: 28672 x 4096
// 36.1 / 32.3 us, 32768 x 4096 40.9 / 34.3, 10261 x 16384 48.0 / 43.1, 13824 x 8192 30.8 / 30.4; 28672 x 4096 from the cache 26.2 / 27.3), costs at others (37888 x
// 3584 35.0 / 38.0, 28160 x 4352 33.1 / 37.5, 18944 x 7168 35.2 / 38.0, 20949 x 5003 36.0 / 38.8, 4352 x 28672 33.5 / 34.2) and in smaller ones (4096 x 8192
// 10.5 / 11.2).  Of 57 widths at 120 MB one other gained, 11008 (39.5 / 34.9), its neighbours 10752 and 11264 not.
// STREAM: integers of more than 192 MB, of which the last-level cache keeps more if the packed weights go past it (cached / streamed, from HBM and
// again at once: 35882 x 7168 74.4 / 69.3 and 73.4 / 54.6, 29290 x 7168, 200 MB, 57.0 / 57.0 and 54.0 / 46.7, but 26304 x 7168, 180 MB, 48.0 / 51.6 and 46.3 / 40.5).
constexpr int PACK_TILES = 4;

template <bool ALONG_K, bool STREAM>
__global__ __launch_bounds__(256) void pack_weights_kernel(const int8_t *__restrict__ w, int64_t N, int64_t K, int64_t row_blocks, int64_t tile_groups,
                                                           uint8_t *__restrict__ out)
{
    const int64_t row_block = ALONG_K ? blockIdx.x / tile_groups : blockIdx.x % row_blocks;
    const int64_t tile_group = ALONG_K ? blockIdx.x % tile_groups : blockIdx.x / row_blocks;
    const int64_t row = row_block * 64 + (threadIdx.x >> 2);
    const int64_t tile0 = tile_group * PACK_TILES, tiles = k_tiles(K);
    const int c = threadIdx.x & 3;                 // granule inside the 64-byte segment
    if (row >= N) return;
    const int8_t *src = w + row * K;
    uint4 v[PACK_TILES][2];
#pragma unroll
    for (int i = 0; i < PACK_TILES; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) v[i][h] = load_row16(src, (tile0 + i) * KT + c * 32 + h * 16, K);     // K padding is zero
#pragma unroll
    for (int i = 0; i < PACK_TILES; ++i)
        if (tile0 + i < tiles) {
            const v4i p = {(int)pack8(v[i][0].x, v[i][0].y), (int)pack8(v[i][0].z, v[i][0].w), (int)pack8(v[i][1].x, v[i][1].y), (int)pack8(v[i][1].z, v[i][1].w)};
            v4i *const dst = reinterpret_cast<v4i *>(out + ((tile0 + i) * N + row) * SEG + c * 16);
            if (STREAM) __builtin_nontemporal_store(p, dst);
            else *dst = p;
        }
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t *__restrict__ packed, int64_t rows, int64_t K,
                                                     int8_t *__restrict__ out)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * K) return;
    int64_t row = idx / K, k = idx % K;
    uint8_t b = packed[((k / KT) * rows + row) * SEG + (k % KT) / 2];
    int v = (k & 1) ? (b >> 4) : (b & 15);
    out[idx] = (int8_t)(v >= 8 ? v - 16 : v);
}

// acc[t][o] = sum_k q[t][k] * w[o][k], straight from the packed buffers with the 8-way INT4 dot
// instruction; one thread per output.  Also the library's answer for shapes nothing else covers.
__global__ __launch_bounds__(256) void linear_ref_kernel(const uint8_t *__restrict__ xq, const uint8_t *__restrict__ wq,
                                                         int64_t M, int64_t N, int64_t ktiles, float s_a,
                                                         const float *__restrict__ s_w, const float *__restrict__ d, int zp,
                                                         const int32_t *__restrict__ wsum, uint16_t *__restrict__ y,
                                                         int32_t *__restrict__ acc_out)
{
    const int64_t blocks_n = (N + 15) / 16;
    int64_t o = ((int64_t)blockIdx.x % blocks_n) * 16 + (threadIdx.x & 15);
    int64_t t = ((int64_t)blockIdx.x / blocks_n) * 16 + (threadIdx.x >> 4);
    if (o >= N || t >= M) return;
    int acc = 0;
    for (int64_t kt = 0; kt < ktiles; ++kt) {
        const uint4 *a = reinterpret_cast<const uint4 *>(xq + (kt * M + t) * SEG);
        const uint4 *b = reinterpret_cast<const uint4 *>(wq + (kt * N + o) * SEG);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint4 av = a[c], bv = b[c];
            acc = __builtin_amdgcn_sdot8((int)av.x, (int)bv.x, acc, false);
            acc = __builtin_amdgcn_sdot8((int)av.y, (int)bv.y, acc, false);
            acc = __builtin_amdgcn_sdot8((int)av.z, (int)bv.z, acc, false);
            acc = __builtin_amdgcn_sdot8((int)av.w, (int)bv.w, acc, false);
        }
    }
    float cw = s_a * s_w[o];
    y[t * N + o] = dequant_bf16(remove_zero_point(acc, zp, wsum, o), cw, d, t);
    if (acc_out) acc_out[t * N + o] = acc;          // the raw accumulator sum_k v w
}

hipError_t launch_pack_weights(const int8_t *w, int64_t N, int64_t K, uint8_t *out, hipStream_t s)
{
    const int64_t row_blocks = (N + 63) / 64, tile_groups = (k_tiles(K) + PACK_TILES - 1) / PACK_TILES, blocks = row_blocks * tile_groups;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(256);
    const bool along_k = K % 4096 == 0 && K <= 16384 && N * K >= (int64_t)108 << 20, stream = N * K > (int64_t)192 << 20;
#define FPTQ_PACK(ALONG_K, STREAM) pack_weights_kernel<ALONG_K, STREAM><<<grid, block, 0, s>>>(w, N, K, row_blocks, tile_groups, out)
    if (along_k)
        stream ? FPTQ_PACK(true, true) : FPTQ_PACK(true, false);
    else
        stream ? FPTQ_PACK(false, true) : FPTQ_PACK(false, false);
#undef FPTQ_PACK
    return hipGetLastError();
}

hipError_t launch_unpack(const uint8_t *packed, int64_t rows, int64_t K, int8_t *out, hipStream_t s)
{
    int64_t blocks = (rows * K + 255) / 256;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    unpack_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(packed, rows, K, out);
    return hipGetLastError();
}

// sum_k w[o][k] per output channel (what an activation zero point multiplies); one wave per row, four 16-byte loads in flight
// per lane.  28672 x 4096: 17 us behind the packer, which leaves part of the matrix in the last-level cache; a byte per
// load took 83.
__global__ __launch_bounds__(256) void weight_row_sums_kernel(const int8_t *__restrict__ w, int64_t N, int64_t K,
                                                              int32_t *__restrict__ sums)
{
    const int lane = threadIdx.x & 63;
    const int64_t o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (o >= N) return;
    const int8_t *row = w + o * K;
    int s = 0;
    for (int64_t k0 = (int64_t)lane * 16; k0 < K; k0 += 4 * 1024) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load_row16(row, k0 + u * 1024, K);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            s = __builtin_amdgcn_sdot4((int)v[u].x, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)v[u].y, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)v[u].z, 0x01010101, s, false);
            s = __builtin_amdgcn_sdot4((int)v[u].w, 0x01010101, s, false);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) sums[o] = s;
}

hipError_t launch_weight_row_sums(const int8_t *w, int64_t N, int64_t K, int32_t *sums, hipStream_t s)
{
    int64_t blocks = (N + 3) / 4;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    weight_row_sums_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(w, N, K, sums);
    return hipGetLastError();
}

hipError_t launch_linear_ref(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                             const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                             hipStream_t s)
{
    int64_t blocks = ((N + 15) / 16) * ((M + 15) / 16);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    linear_ref_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(xq, wq, M, N, k_tiles(K), s_a, s_w, d, zp, wsum, y, acc);
    return hipGetLastError();
}

}  // namespace fptq
