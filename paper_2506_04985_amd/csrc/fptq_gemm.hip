// Prefill kernel of the quantized linear layer: INT4 x INT4 matmul on the INT8 matrix cores with
// INT32 accumulation, and the float-scale epilogue to bf16 (App. J and App. B of the paper).
//
// CDNA4 has no 4-bit integer MFMA, so nibbles are widened to bytes in registers just before
// v_mfma_i32_32x32x32_i8.  A packed dword p holds 8 nibbles; (p << 4) & 0xF0F0F0F0 and
// p & 0xF0F0F0F0 are 2 x 4 signed bytes equal to 16 * value (the nibble's sign bit lands on the
// byte's sign bit).  Both operands are widened the same way, so the accumulator holds exactly
// 256 * acc: |acc| <= 64 K keeps 256 * acc inside int32 for K up to 131071, and the epilogue
// shifts it back.  Which k lands in which byte of an operand does not matter as long as both
// operands agree, and they do: the same code widens the same byte offsets of X and W.
//
// Data flow: packed tiles (rows x 64 bytes per K tile, contiguous in HBM) -> LDS by buffer loads
// that write LDS directly (no VGPR staging; rows past the end read as zero through the buffer
// descriptor's bounds check), STAGES-deep ring, one barrier per K tile -> ds_read_b128 fragments
// -> widen -> MFMA.  The 16-byte granules of a row are XOR-swizzled in LDS so that the fragment
// reads are bank-conflict free.
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "fptq_common.h"

namespace fptq {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int MAX_SPLITS = 4;     // K ranges per output tile in the split-K variant
constexpr int SPLIT_COUNTERS = 1024;   // arrival counters at the start of a split-K workspace (one per output tile)

// OCC_ = workgroups meant to share a CU (caps the register budget: 512 / OCC_ per lane).  KS_ = K groups:
// KS_ sets of WAVES waves work on the same output tile, set g on K tiles g, g + KS_, ..., each with its own
// LDS ring; their accumulators are added through LDS and every group runs its share of the epilogue.  A
// problem with at most one workgroup per CU runs one wave per SIMD, which cannot hide its own LDS and VALU
// latencies; more K groups give every SIMD more waves without needing more output tiles.
// SPLIT_: several workgroups share an output tile, each on a contiguous range of K tiles; they leave their
// partial accumulators in a caller-provided workspace and the last one to arrive adds them and runs the epilogue.
template <int WAVES_N_, int WAVES_M_, int TN_, int TM_, int STAGES_, int OCC_ = 1, int KS_ = 1, bool SPLIT_ = false>
struct GemmCfg {
    static constexpr int WAVES_N = WAVES_N_, WAVES_M = WAVES_M_, TN = TN_, TM = TM_, STAGES = STAGES_, OCC = OCC_, KS = KS_;
    static constexpr bool SPLIT = SPLIT_;
    static constexpr int ACC_REGS = TN_ * TM_ * 16;             // accumulator registers of a lane
    static constexpr int BN = WAVES_N * TN * 32, BM = WAVES_M * TM * 32;
    static constexpr int WAVES = WAVES_N * WAVES_M, THREADS = 64 * WAVES * KS;
    static constexpr int W_BYTES = BN * SEG, X_BYTES = BM * SEG, STAGE_BYTES = W_BYTES + X_BYTES;
    // every wave copies a contiguous run of rows of each operand tile, 1 KB (16 rows) per load
    static constexpr int W_LOADS = W_BYTES / (WAVES * 1024), X_LOADS = X_BYTES / (WAVES * 1024);
    static constexpr int LOADS = W_LOADS + X_LOADS;
    static constexpr int RING_BYTES = STAGES * STAGE_BYTES, LDS_BYTES = KS * RING_BYTES;
    static_assert(W_BYTES % (WAVES * 1024) == 0 && X_BYTES % (WAVES * 1024) == 0, "tile must split over waves");
    static_assert(W_LOADS >= 1 && W_LOADS <= 4 && X_LOADS >= 1 && X_LOADS <= 4, "the fill schedule issues at most two chunks per quarter");
    // A K tile's fill goes in quarters: W chunk q and X chunk q (KS = 1), or two W chunks, two X chunks, the other W chunks, the other X chunks: loads of
    // adjacent lines side by side, and one LDS base for both.
    static constexpr int W_FIRST = W_LOADS < 2 ? W_LOADS : 2, X_FIRST = X_LOADS < 2 ? X_LOADS : 2, HALF_LOADS = W_FIRST + X_FIRST;      // quarters 0 and 1
    // Steps in the unrolled loop, so that the sets of descriptors and (KS > 1) the ring positions are known at compile time.  A wave alone on its SIMD waits
    // for every instruction, and of the 190 that a 64 x 64 block took per K tile, 55 were scalar ones for addresses; now 155.  A wave of these launches turns
    // the loop a few times only (twice at 256 x 2048 x 8192 in two K ranges), so it is bound by how fast code arrives as well, and that differs from card to card.
    // The steps that are left after the last whole turn are therefore the loop's own, each behind a test, and not copies behind the loop, which cost time even
    // where none is taken.  us, rolled / copies behind the loop / tests in it, on a card where code arrives fast and on one where it arrives slowly:
    //     256 x 2048 x 8192, with its quantizer   13.4 / 12.4 / 12.5,  13.8 / 14.5 / 13.5     96 x 28672 x 4096, weights from HBM   17.8 / 18.7 / 17.1,  19.1 / 20.0 / 18.7
    //     1000 x 4096 x 4096, weights from HBM    17.6 / 16.2 / 16.6,  18.0 / 21.6 / 17.6     512 x 8192 x 8192, weights from HBM   31.9 / 28.5 / 29.3,  33.0 / 30.6 / 30.7
    // of 32 launches on three cards none is slower than rolled by more than 1 %.  Six steps, with two sets of descriptors instead of three: up to 11 % slower
    // from HBM (100 x 30000 x 3000 16.4, 18.1; three steps 15.9).  The 256 x 256 tile would spill.
    static constexpr int UNROLL = ACC_REGS == 256 ? 1 : KS == 1 ? 2 : STAGES;
    static_assert(STAGES >= 3, "pipeline needs three stages");
    static_assert(TN <= 4, "a wave's channel run must fit 16 lanes of 8 channels in the epilogue");
    // After the K loop the K groups exchange accumulators so that each ends up with the sum of SUBS of the wave's
    // TN x TM sub-tiles (counted along n first): TNE along n, TME along m.
    static constexpr int SUBS = TN * TM / KS;
    static constexpr int TNE = SUBS >= TN ? TN : SUBS, TME = SUBS >= TN ? SUBS / TN : 1;
    static constexpr int NSC = (TNE * 32 + 63) / 64;           // channel scales a lane fetches for the epilogue
    static_assert(TN * TM % KS == 0 && TNE * TME == SUBS && TN % TNE == 0, "the K groups share the sub-tiles evenly, in runs along n");
    static_assert((KS - 1) * TN * TM * WAVES * 4096 <= LDS_BYTES, "the K groups' accumulators are added through LDS");
};

// widen two packed dwords (16 nibbles) into one MFMA operand of 16 bytes, each 16 * value
__device__ inline v4i widen(int p0, int p1)
{
    v4i o;
    o.x = (p0 << 4) & (int)0xF0F0F0F0;
    o.y = p0 & (int)0xF0F0F0F0;
    o.z = (p1 << 4) & (int)0xF0F0F0F0;
    o.w = p1 & (int)0xF0F0F0F0;
    return o;
}

// One 1 KB chunk (16 rows) of an operand tile, HBM -> LDS.  J is the chunk number inside the run of
// chunks this wave copies: the immediate offset (a compile-time constant of the instruction)
// advances the HBM and the LDS address together, so all chunks share one VGPR offset and one LDS base.
template <int J>
__device__ inline void load_chunk(__amdgpu_buffer_rsrc_t r, uint8_t *lds_base, int voff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, LDS_PTR(lds_base), 16, voff, 0, J * 1024, 0);
}

// Channel scales (and, with a zero point, the weight row sums) of a run of TNE * 32 channels, one or two per lane.
template <int TNE, bool ZP>
__device__ inline void load_scales(float (&scv)[(TNE * 32 + 63) / 64], int32_t (&zwv)[(TNE * 32 + 63) / 64],
                                   const float *__restrict__ s_w, const int32_t *__restrict__ wsum, int nw0, int N, int lane)
{
#pragma unroll
    for (int i = 0; i < (TNE * 32 + 63) / 64; ++i) {
        const int n = min(nw0 + min(lane + 64 * i, TNE * 32 - 1), N - 1);
        scv[i] = s_w[n];
        zwv[i] = ZP ? wsum[n] : 0;
    }
}

// What a wave does with its finished sub-tiles a[t][i] (t < TNE along n from channel nw0, i < TME along m from
// token mw0; sub-tile numbers sub0 .. of the wave's TN x TM, counted along n first): the split-K exchange, then
// the epilogue.
template <class C, int TNE, int TME, int STORE, bool DUMP, bool ZP>
__device__ inline void finish(v16i (&a)[TNE][TME], const float (&scv)[(TNE * 32 + 63) / 64],
                              const int32_t (&zwv)[(TNE * 32 + 63) / 64], uint8_t *lds, int wave_all, int wave, int lane,
                              int sub0, int nw0, int mw0, int M, int N, float s_a, const float *__restrict__ d, int zp,
                              const int32_t *__restrict__ wsum, uint16_t *__restrict__ y, int32_t *__restrict__ acc_out,
                              int32_t *ws, int splits, int split, int pid, int total)
{
    const int fi = lane & 31, fg = lane >> 5;
    // ---- split K: leave the partial tile in the workspace, count the arrival, and let the last workgroup of
    // the tile add the others' partials and go on to the epilogue.  Nobody waits for anybody, so there is nothing
    // to hang on.  The workgroups of a tile run on different XCDs, whose L2s are not coherent with each other, and
    // a device-wide fence would write back and invalidate a whole L2 per workgroup; instead the partials are
    // stored and loaded with the device-coherent cache policy (sc0 sc1: written through to, and read from, the
    // memory side), the stores are complete (vmcnt) before the arrival is counted, and the count is an atomic
    // at the same scope.  Workspace: SPLIT_COUNTERS arrival counters (zero between calls; the first `total` are used:
    // a region of fixed size, so that calls of different shapes that share a workspace agree on where it ends), then
    // [splits][total][sub-tile][quad][threads of a K group] partials as 16-byte quads, lane-contiguous.
    if (C::SPLIT) {
        constexpr int TPG = C::WAVES * 64, COHERENT = 1 | 16;     // aux bits: sc0, sc1
        const int64_t slice = (int64_t)C::ACC_REGS * TPG;
        int32_t *counters = ws, *parts = ws + SPLIT_COUNTERS;
        int *flag = reinterpret_cast<int *>(lds + C::LDS_BYTES - 16);     // clear of the epilogue's patches
        const int qoff = (wave * 64 + lane) * 16 + sub0 * (4 * TPG * 16);
        const __amdgpu_buffer_rsrc_t mine = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(parts + ((int64_t)split * total + pid) * slice), 0, (int)slice * 4, RSRC_FLAGS);
#pragma unroll
        for (int i = 0; i < TME; ++i)
#pragma unroll
            for (int t = 0; t < TNE; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4i v = {a[t][i][4 * q], a[t][i][4 * q + 1], a[t][i][4 * q + 2], a[t][i][4 * q + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(v, mine, qoff + ((i * TNE + t) * 4 + q) * (TPG * 16), 0, COHERENT);
                }
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // this wave's partials have reached the memory side
        __syncthreads();
        if (threadIdx.x == 0) *flag = __hip_atomic_fetch_add(counters + pid, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*flag != splits - 1) return;             // the whole workgroup: not the last one of this tile
        // the other (at most MAX_SPLITS - 1) partial tiles, read side by side so that their latencies overlap
        __amdgpu_buffer_rsrc_t other[MAX_SPLITS - 1];
#pragma unroll
        for (int j = 0; j < MAX_SPLITS - 1; ++j) {
            const int s2 = (split + 1 + j) % splits;            // j < splits - 1: every other split once
            other[j] = __builtin_amdgcn_make_buffer_rsrc((void *)(parts + ((int64_t)s2 * total + pid) * slice), 0,
                                                         j < splits - 1 ? (int)slice * 4 : 0, RSRC_FLAGS);
        }
#pragma unroll
        for (int i = 0; i < TME; ++i)
#pragma unroll
            for (int t = 0; t < TNE; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v4i v[MAX_SPLITS - 1];
#pragma unroll
                    for (int j = 0; j < MAX_SPLITS - 1; ++j)      // an empty descriptor (j >= splits - 1) reads zeros
                        v[j] = __builtin_amdgcn_raw_buffer_load_b128(other[j], qoff + ((i * TNE + t) * 4 + q) * (TPG * 16), 0, COHERENT);
#pragma unroll
                    for (int j = 0; j < MAX_SPLITS - 1; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[t][i][4 * q + e] += v[j][e];
                }
        if (threadIdx.x == 0) counters[pid] = 0;     // as it was found, for the next call
    }

    // ---- epilogue.  W was the A operand, so an accumulator tile is [n][m]: a lane owns token
    // m = lane % 32 and, per register quad q, four consecutive output channels
    // n = 8 q + 4 (lane / 32) + (r % 4).  The register holds 256 * acc; (float)(256 * acc) equals
    // 256 * (float)acc exactly (acc has fewer than 24 significant bits), and the 2^-8 is folded into
    // the channel scale, which is exact as well, so y = bf16((float)acc * (s_a * s_w[n]) [* d_t]) to
    // the bit.  Bound by latencies where a CU has one workgroup, so constants are read once and a group of 32 tokens is read back while the next
    // one is computed.  The halves of a wave exchange quads, so that a lane holds eight consecutive channels; those 16 bytes go through
    // a wave-private LDS patch ([32 tokens][TNE * 32 channels], the granules of a row permuted so that eight lanes hit different banks
    // both ways), so that HBM sees whole row segments.
    constexpr int WN = TNE * 32, ROW_BYTES = WN * 2;          // this wave's run of channels
    constexpr int GRANULES = WN / 8;                          // 16-byte pieces of a row
    // With an activation zero point z the sum wanted is sum_k (v - z) w = acc - z * wsum[n]; the
    // correction is staged as 256 * z * wsum[n] next to the scales (|.| < 2^31 for K <= 65535).
    constexpr int WAVE_LDS = 32 * ROW_BYTES + WN * 8;
    uint8_t *const patch = lds + wave_all * WAVE_LDS;
    float *const cwbuf = reinterpret_cast<float *>(patch + 32 * ROW_BYTES);
    int32_t *const zwbuf = reinterpret_cast<int32_t *>(cwbuf + WN);
    float dm[TME];
#pragma unroll
    for (int tm = 0; tm < TME; ++tm) dm[tm] = d ? d[min(mw0 + tm * 32 + fi, M - 1)] : 1.0f;
#pragma unroll
    for (int i = 0; i < (WN + 63) / 64; ++i) {
        const int c = lane + 64 * i;
        if (c < WN) {
            cwbuf[c] = (s_a * scv[i]) * 0.00390625f;
            if (ZP) zwbuf[c] = (zp * zwv[i]) * 256;
        }
    }
    auto in_order = [] {       // a wave's LDS operations complete in order: only the compiler has to be kept from exchanging them
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    in_order();
    float4 cw[TNE][4];
#pragma unroll
    for (int tn = 0; tn < TNE; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) cw[tn][q] = *reinterpret_cast<const float4 *>(cwbuf + tn * 32 + 8 * q + 4 * fg);
    // granule g of row r lies in slot g ^ turn(r)
    auto turn = [](int r) { return GRANULES % 8 == 0 ? r & 7 : (r >> 2) & 3; };
    auto to_lds = [&](int tm) {
        uint8_t *const to = patch + fi * ROW_BYTES;
        const int slot = fg ^ turn(fi);
#pragma unroll
        for (int tn = 0; tn < TNE; ++tn)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint32_t p[2][2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4 c4 = cw[tn][2 * j + q];
                    const float c[4] = {c4.x, c4.y, c4.z, c4.w};
                    const int r0 = 8 * j + 4 * q;
                    int32_t a4[4] = {a[tn][tm][r0], a[tn][tm][r0 + 1], a[tn][tm][r0 + 2], a[tn][tm][r0 + 3]};
                    if (ZP) {
                        const int4 z4 = *reinterpret_cast<const int4 *>(zwbuf + tn * 32 + 2 * r0 + 4 * fg);
                        a4[0] -= z4.x, a4[1] -= z4.y, a4[2] -= z4.z, a4[3] -= z4.w;
                    }
                    float yf[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) yf[e] = (float)a4[e] * c[e] * dm[tm];
                    p[q][0] = pack_bf16(yf[0], yf[1]), p[q][1] = pack_bf16(yf[2], yf[3]);
                }
                // lanes 32 .. 63 of the first and 0 .. 31 of the second change places: quads 2 j of both halves, and 2 j + 1
                const auto lo = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
                *reinterpret_cast<uint4 *>(to + ((tn * 4 + 2 * j) ^ slot) * 16) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
            }
        in_order();
    };
    // read back as row segments: 16 bytes (8 channels) per lane, GRANULES lanes per token row (rounded up to a power of two; the surplus lanes idle)
    constexpr int LANES_PER_ROW = GRANULES <= 4 ? 4 : GRANULES <= 8 ? 8 : 16, ROWS_PER_PASS = 64 / LANES_PER_ROW, PASSES = 32 / ROWS_PER_PASS;
    const int row = lane / LANES_PER_ROW, col = lane % LANES_PER_ROW, nn = nw0 + col * 8;
    const bool live = col < GRANULES && nn < N;
    // an offset past every descriptor's end for what is not to be stored; rows past M fail the descriptor's check
    const uint32_t row_stride = (uint32_t)N * 2;
    const uint32_t y_off = live && (STORE != ANY_ALIGNMENT || nn + 8 <= N) ? (uint32_t)row * row_stride + (uint32_t)nn * 2 : 0x80000000u;
    to_lds(0);
#pragma unroll
    for (int tm = 0; tm < TME; ++tm) {
        const int mt0 = mw0 + tm * 32;
        const int m = mt0 + fi;
        uint4 v[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int r = p * ROWS_PER_PASS + row;
            v[p] = *reinterpret_cast<const uint4 *>(patch + r * ROW_BYTES + ((GRANULES == LANES_PER_ROW ? col : min(col, GRANULES - 1)) ^ turn(r)) * 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (tm + 1 < TME) to_lds(tm + 1);
        store_rows<STORE, PASSES, ROWS_PER_PASS>(v, y, y_off, mt0, row, nn, live, M, N, nw0 + WN > N);
        if (DUMP) {      // parity dump of the integer accumulators (never a timed path)
#pragma unroll
            for (int tn = 0; tn < TNE; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int n = nw0 + tn * 32 + 8 * q + 4 * fg + e;
                        if (m < M && n < N) acc_out[(int64_t)m * N + n] = a[tn][tm][4 * q + e] >> 8;
                    }
        }
    }
}

// ZP: the epilogue removes an activation zero point (wsum is then non-null); a separate instance, so that the symmetric
// grid's epilogue carries neither its code nor its registers (the 256 x 256 instance spilled 13 registers with both in one).  Of the instances
// that calls without accumulators run, only that tile's use scratch, once per tile: 12 registers where N % 8 != 0, 16 with a zero point there, 1 with one
// elsewhere (4096 x 8193 x 1024 56.1 us, with the old epilogue and no scratch 60.5; with a zero point 59.9 and 62.8).
template <class C, int STORE, bool DUMP, bool ZP>
__global__ __launch_bounds__(C::THREADS, C::OCC) void linear_mfma_kernel(
    const uint8_t *__restrict__ xq, const uint8_t *__restrict__ wq, int M, int N, int ktiles, int tiles_m,
    int tiles_n, float s_a, const float *__restrict__ s_w, const float *__restrict__ d, int zp,
    const int32_t *__restrict__ wsum, uint16_t *__restrict__ y, int32_t *__restrict__ acc_out, int32_t *ws, int splits, int map_mode)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = C::KS > 1 ? wave_all / C::WAVES : 0, wave = C::KS > 1 ? wave_all % C::WAVES : wave_all;   // K group, wave in it
    const int wave_n = wave % C::WAVES_N, wave_m = wave / C::WAVES_N;
    uint8_t *const ring = lds + kg * C::RING_BYTES;                      // this K group's LDS ring

    // ---- tile of this workgroup.  Workgroups are dealt round-robin to the 8 XCDs; give each XCD a
    // contiguous run of logical tiles so that its L2 sees neighbouring tiles, then walk the tile grid
    // in bands of 8 N-tiles with M fastest, so that concurrent tiles share X and W panels.
    const int total = tiles_m * tiles_n;
    int pid = blockIdx.x, split = 0;
    if (C::SPLIT) {                                  // workgroup = (split, tile), tiles fastest
        split = pid / total;
        pid -= split * total;
    }
    if (map_mode == 0) {                             // (map_mode 1, a measurement aid: tiles dealt round-robin to the XCDs as they come)
        const int per = (total + 7) / 8, tall = total % 8 == 0 ? 8 : total % 8;
        const int xcd = pid % 8, local = pid / 8;
        pid = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
    }
    constexpr int GN = 8;
    const int band = pid / (GN * tiles_m), in_band = pid % (GN * tiles_m);
    const int band_w = min(GN, tiles_n - band * GN);
    const int bn = band * GN + in_band % band_w, bm = in_band / band_w;
    const int n0 = bn * C::BN, m0 = bm * C::BM;

    // ---- global -> LDS copy plan.  One K tile of an operand is rows x 64 bytes, contiguous in HBM,
    // and its LDS image has the same linear layout except that the four 16-byte granules of a row
    // are permuted: LDS slot s of a row holds granule s ^ swz(row), swz(row) = (row >> 2) & 3.
    // (A ds_read_b128 is served 16 lanes at a time; the 16 rows they read then fall into 16
    // different 16-byte bank groups: address bits 7:4 = (row % 4) * 4 + slot.)
    // A wave-level load fills 1 KB: lane l lands at byte 16 l, i.e. row l / 4, slot l % 4, and the
    // row's swizzle is (l / 16) & 3 for every 16-row chunk.  Each wave copies W_LOADS (X_LOADS)
    // consecutive chunks, addressed by one VGPR offset plus 1 KB immediates, which move the HBM
    // and the LDS address together.
    const int lane_src = (lane >> 2) * SEG + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
    const int w_voff = (n0 + wave * (C::W_LOADS * 16)) * SEG + lane_src;
    const int x_voff = (m0 + wave * (C::X_LOADS * 16)) * SEG + lane_src;
    const int w_lds0 = wave * (C::W_LOADS * 1024), x_lds0 = C::W_BYTES + wave * (C::X_LOADS * 1024);
    const int64_t w_slab = (int64_t)N * SEG, x_slab = (int64_t)M * SEG;   // bytes per K tile of all rows

    // per-slab descriptors: rows past N (M) fail the bounds check and read as zero.  Step j of this K group
    // is K tile kt_begin + j * KS + kg; a step past the last tile gets an empty descriptor, so its loads are still
    // issued (the outstanding-load count stays uniform) but read nothing and land as zeros.  The steps are asked for in order, so that
    // an addition makes the next addresses.
    int kt_begin = 0, kt_end = ktiles;               // K tiles of this workgroup
    if (C::SPLIT) {
        const int per = (ktiles + splits - 1) / splits;
        kt_begin = split * per;
        kt_end = min(ktiles, kt_begin + per);
    }
    const uint8_t *w_next = wq + (kt_begin + kg) * w_slab, *x_next = xq + (kt_begin + kg) * x_slab;
    int tiles_left = kt_end - kt_begin - kg;
    const int64_t w_step = C::KS * w_slab, x_step = C::KS * x_slab;
    auto next_descs = [&](__amdgpu_buffer_rsrc_t &w, __amdgpu_buffer_rsrc_t &x) {
        w = __builtin_amdgcn_make_buffer_rsrc((void *)w_next, 0, tiles_left > 0 ? (int)w_slab : 0, RSRC_FLAGS);
        x = __builtin_amdgcn_make_buffer_rsrc((void *)x_next, 0, tiles_left > 0 ? (int)x_slab : 0, RSRC_FLAGS);
        w_next += w_step, x_next += x_step, tiles_left -= C::KS;
    };
    // quarter q (0..3) of the fill of one K tile
    auto chunk = [&](auto which, __amdgpu_buffer_rsrc_t r, uint8_t *base, int voff, int loads) {
        if (decltype(which)::value < loads) load_chunk<decltype(which)::value>(r, base, voff);
    };
    auto fill_quarter = [&](__amdgpu_buffer_rsrc_t wr, __amdgpu_buffer_rsrc_t xr, int stage, int q) {
        const std::integral_constant<int, 0> c0;
        const std::integral_constant<int, 1> c1;
        const std::integral_constant<int, 2> c2;
        const std::integral_constant<int, 3> c3;
        uint8_t *const wb = ring + stage * C::STAGE_BYTES + w_lds0, *const xb = ring + stage * C::STAGE_BYTES + x_lds0;
        if constexpr (C::KS == 1) {
            if (q == 0) chunk(c0, wr, wb, w_voff, C::W_LOADS), chunk(c0, xr, xb, x_voff, C::X_LOADS);
            if (q == 1) chunk(c1, wr, wb, w_voff, C::W_LOADS), chunk(c1, xr, xb, x_voff, C::X_LOADS);
            if (q == 2) chunk(c2, wr, wb, w_voff, C::W_LOADS), chunk(c2, xr, xb, x_voff, C::X_LOADS);
            if (q == 3) chunk(c3, wr, wb, w_voff, C::W_LOADS), chunk(c3, xr, xb, x_voff, C::X_LOADS);
        } else {
            if (q == 0) chunk(c0, wr, wb, w_voff, C::W_LOADS), chunk(c1, wr, wb, w_voff, C::W_LOADS);
            if (q == 1) chunk(c0, xr, xb, x_voff, C::X_LOADS), chunk(c1, xr, xb, x_voff, C::X_LOADS);
            if (q == 2) chunk(c2, wr, wb, w_voff, C::W_LOADS), chunk(c3, wr, wb, w_voff, C::W_LOADS);
            if (q == 3) chunk(c2, xr, xb, x_voff, C::X_LOADS), chunk(c3, xr, xb, x_voff, C::X_LOADS);
        }
    };

    // ---- fragment read plan: lane (i = lane % 32, g = lane / 32) of a 32-row sub-tile reads, for
    // K half kk, granule 2 kk + g of row i (one ds_read_b128): its low 8 bytes feed the first MFMA
    // step of the half, the high 8 bytes the second.  Sub-tile bases are multiples of 32 rows, so
    // the swizzle depends on the lane only.
    const int fi = lane & 31, fg = lane >> 5;
    int frag_off[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) frag_off[kk] = fi * SEG + (((2 * kk + fg) ^ ((fi >> 2) & 3)) << 4);
    const int w_wave = wave_n * (C::TN * 32 * SEG), x_wave = C::W_BYTES + wave_m * (C::TM * 32 * SEG);

    v16i acc[C::TN][C::TM];
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tn][tm][r] = 0;

    // ---- software pipeline.
    // A K tile is four MFMA steps of 32 values, i.e. four groups G0..G3 of TN*TM MFMAs.  One
    // ds_read_b128 per operand row brings two steps (R0: steps 0-1, R1: steps 2-3).  While the
    // MFMAs of step s run, the operands of step s+1 are widened (3 VALU per MFMA), the next batch of
    // fragment reads is issued one read every other MFMA, and the HBM->LDS fill of a later tile is
    // issued a quarter per group.  Spreading the LDS reads and the fill matters: the four waves run
    // in lock step, and a burst of either backs up the LDS / address queues and stalls MFMA issue.
    //   G0(kt): MFMA step 0 | widen step 1 (R0 high)  | read R1(kt)     | fill(kt+S-1) quarter 2
    //   G1(kt): MFMA step 1 | widen step 2 (R1 low)   |                 | fill(kt+S-1) quarter 3
    //   -- tile kt+1 has landed; barrier; every wave is done reading tile kt --
    //   G2(kt): MFMA step 2 | widen step 3 (R1 high)  | read R0(kt+1)   | fill(kt+S) quarter 0, into tile kt's buffer
    //   G3(kt): MFMA step 3 | widen step 0' (R0' low) |                 | fill(kt+S) quarter 1
    v4i opW[2][C::TN], opX[2][C::TM], rawW[2][C::TN], rawX[2][C::TM];
    auto read_frags = [&](int stage, int kk, v4i (&wraw)[C::TN], v4i (&xraw)[C::TM]) {
        const uint8_t *wb = ring + stage * C::STAGE_BYTES + w_wave + frag_off[kk];
        const uint8_t *xb = ring + stage * C::STAGE_BYTES + x_wave + frag_off[kk];
#pragma unroll
        for (int tn = 0; tn < C::TN; ++tn) wraw[tn] = *reinterpret_cast<const v4i *>(wb + tn * (32 * SEG));
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm) xraw[tm] = *reinterpret_cast<const v4i *>(xb + tm * (32 * SEG));
    };
    // MFMAs on the current operands, widening half h of the raw fragments into the next operands
    auto group = [&](const v4i (&cw)[C::TN], const v4i (&cx)[C::TM], v4i (&nw)[C::TN], v4i (&nx)[C::TM],
                     const v4i (&rw)[C::TN], const v4i (&rx)[C::TM], int h) {
        constexpr int NM = C::TN * C::TM, NOP = C::TN + C::TM;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int tn = i / C::TM, tm = i % C::TM;
            acc[tn][tm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cw[tn], cx[tm], acc[tn][tm], 0, 0, 0);
#pragma unroll
            for (int o = (i * NOP) / NM; o < ((i + 1) * NOP) / NM; ++o) {   // spread the NOP widenings over the NM MFMAs
                if (o == 0) nw[0] = widen(rw[0][2 * h], rw[0][2 * h + 1]);    // order: W0, X0..X(TM-1), W1..W(TN-1)
                else if (o <= C::TM) nx[o - 1] = widen(rx[o - 1][2 * h], rx[o - 1][2 * h + 1]);
                else nw[o - C::TM] = widen(rw[o - C::TM][2 * h], rw[o - C::TM][2 * h + 1]);
            }
        }
    };
    // pin the interleave of one group: one MFMA, then its share of VALU work; an LDS read after
    // the MFMAs that are followed by a widening when the group issues reads; the fill loads of
    // quarter q in the middle
    auto pin = [&](bool reads, int q) {
        constexpr int NM = C::TN * C::TM, NOP = C::TN + C::TM, VPM = (6 * NOP + NM - 1) / NM;
        const int n_vmem = C::KS == 1 ? (q < C::W_LOADS ? 1 : 0) + (q < C::X_LOADS ? 1 : 0)
                                      : q == 0 ? C::W_FIRST : q == 1 ? C::X_FIRST : q == 2 ? C::W_LOADS - C::W_FIRST : C::X_LOADS - C::X_FIRST;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (reads) {
#pragma unroll
                for (int o = (i * NOP) / NM; o < ((i + 1) * NOP) / NM; ++o) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            if ((i == NM / 4 && n_vmem > 0) || (i == (3 * NM) / 4 && n_vmem > 1)) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // K-group shapes serve problems whose whole time is one workgroup's walk through K, and have registers to
    // spare: the epilogue's channel scales are fetched here, so that their latency hides under the first tile's.
    const int sub0 = C::KS > 1 ? kg * C::SUBS : 0;                          // first sub-tile of this wave's share of the epilogue
    const int fin_nw0 = n0 + (wave_n * C::TN + sub0 % C::TN) * 32, fin_mw0 = m0 + (wave_m * C::TM + sub0 / C::TN) * 32;
    float scv[C::NSC];
    int32_t zwv[C::NSC];
    if (C::KS > 1) load_scales<C::TNE, ZP>(scv, zwv, s_w, wsum, fin_nw0, N, lane);

    const int steps = (max(kt_end - kt_begin, 0) + C::KS - 1) / C::KS;      // the same for every K group: they share the barriers
#pragma unroll
    for (int s = 0; s < C::STAGES - 1; ++s) {
        __amdgpu_buffer_rsrc_t wr, xr;
        next_descs(wr, xr);
#pragma unroll
        for (int q = 0; q < 4; ++q) fill_quarter(wr, xr, s, q);
    }
    // descriptors of fills
    struct Descs {
        __amdgpu_buffer_rsrc_t w, x;
    } fills[3];      // the one that is half way (step kt+S-1), the one that starts in G2 (step kt+S), and the next
    next_descs(fills[0].w, fills[0].x);
    next_descs(fills[1].w, fills[1].x);
    fill_quarter(fills[0].w, fills[0].x, C::STAGES - 1, 0);
    fill_quarter(fills[0].w, fills[0].x, C::STAGES - 1, 1);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::LOADS * (C::STAGES - 2) + C::HALF_LOADS));   // tile 0 is in
    __builtin_amdgcn_s_barrier();
    read_frags(0, 0, rawW[0], rawX[0]);
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn) opW[0][tn] = widen(rawW[0][tn][0], rawW[0][tn][1]);
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) opX[0][tm] = widen(rawX[0][tm][0], rawX[0][tm][1]);
    __builtin_amdgcn_sched_barrier(0);

    __builtin_amdgcn_s_setprio(2);     // MFMA loop: ahead of other workgroups' prologues and epilogues on this SIMD
    // one K tile, in the ring's position `stage`; a: the fill that is half way, b: the next one, c receives the one after that (unrolled, the sets take turns)
    auto step = [&](int stage, Descs &a, Descs &b, Descs &c) {
        const int stage_next = stage + 1 == C::STAGES ? 0 : stage + 1;
        const int stage_prev = stage == 0 ? C::STAGES - 1 : stage - 1;   // holds tile kt+S-1 (being filled)
        // G0
        read_frags(stage, 1, rawW[1], rawX[1]);
        fill_quarter(a.w, a.x, stage_prev, 2);
        group(opW[0], opX[0], opW[1], opX[1], rawW[0], rawX[0], 1);
        pin(true, 2);
        // G1
        fill_quarter(a.w, a.x, stage_prev, 3);
        group(opW[1], opX[1], opW[0], opX[0], rawW[1], rawX[1], 0);
        pin(false, 3);
        // own loads of tile kt+1 have landed (younger: all of tiles kt+2 .. kt+S-1); the barrier
        // extends that to every wave's loads and says every wave is done reading tile kt
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::LOADS * (C::STAGES - 2)));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        // G2 (after the last tile the fragment reads hit a repeated copy; its results are unused)
        read_frags(stage_next, 0, rawW[0], rawX[0]);
        fill_quarter(b.w, b.x, stage, 0);
        group(opW[0], opX[0], opW[1], opX[1], rawW[1], rawX[1], 1);
        pin(true, 0);
        // G3
        fill_quarter(b.w, b.x, stage, 1);
        if constexpr (C::UNROLL == 1) a = b;
        next_descs(c.w, c.x);
        group(opW[1], opX[1], opW[0], opX[0], rawW[0], rawX[0], 0);
        pin(false, 1);
    };
    int left = steps;
    if constexpr (C::UNROLL == 1) {
        // Counted upwards: downwards from `left` the compiler sets the 256 accumulators twice (4000 x 8200 x 1000 57.4 us, 58.7 with it; 8192 x 8192 x 8192 389 and 394).
        int stage = 0;
        for (int kt = 0; kt < steps; ++kt) {
            step(stage, fills[0], fills[1], fills[1]);
            stage = stage + 1 == C::STAGES ? 0 : stage + 1;
        }
    } else if constexpr (C::UNROLL == 2) {
        auto after = [](int i) { return i + 1 == C::STAGES ? 0 : i + 1; };
        int stage = 0;
        for (; left >= 2; left -= 2) {
            step(stage, fills[0], fills[1], fills[0]);
            step(after(stage), fills[1], fills[0], fills[1]);
            stage = after(after(stage));
        }
        if (left > 0) step(stage, fills[0], fills[1], fills[0]);
    } else {
        constexpr int SETS = C::UNROLL == 3 ? 3 : 2;
        static_assert(C::UNROLL % SETS == 0 && C::UNROLL <= 4, "");
        auto at = [&](int p) { step(p, fills[p % SETS], fills[(p + 1) % SETS], fills[(p + 2) % SETS]); };
        for (; left > 0; left -= C::UNROLL) {
            at(0);
            if (__builtin_expect(left > 1, 1)) at(1);          // falls through: a taken branch per turn (1 % of a launch less than two or three)
            if (__builtin_expect(left > 2, 1)) at(2);
            if constexpr (C::UNROLL == 4) {
                if (__builtin_expect(left > 3, 1)) at(3);
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the tail loads before LDS is reused
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
    __builtin_amdgcn_s_barrier();

    // ---- K groups: the accumulators of the KS groups are added through LDS (integers: exact, order-free) and the
    // sum stays distributed: group g ends up with sub-tiles g * P .. g * P + P - 1 of the wave's TN x TM (counted
    // along n first), so every wave of the workgroup adds 1 / KS of the registers and runs 1 / KS of the epilogue.
    // Every wave first stores the sub-tiles that belong to other groups (16-byte quads, lane-contiguous), then,
    // after one barrier, adds what the others stored for it.
    if (C::KS > 1) {
        constexpr int P = C::SUBS, TPG = C::WAVES * 64, QUAD_BYTES = TPG * 16;
        uint8_t *const xlane = lds + (wave * 64 + lane) * 16;
#pragma unroll
        for (int f = 0; f < C::TN * C::TM; ++f) {
            constexpr int KS1 = C::KS - 1;
            const int h = f / P, p = f % P;                          // receiving group, position in its share
            if (kg != h) {
                const int sender = kg - (kg > h ? 1 : 0);
                uint8_t *dst = xlane + ((h * KS1 + sender) * P + p) * (4 * QUAD_BYTES);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v16i &a = acc[f % C::TN][f / C::TN];
                    *reinterpret_cast<v4i *>(dst + q * QUAD_BYTES) = v4i{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
        __builtin_amdgcn_s_barrier();
        v16i mine[C::TNE][C::TME];
#pragma unroll
        for (int h = 0; h < C::KS; ++h) {
            if (kg == h) {
#pragma unroll
                for (int p = 0; p < P; ++p) mine[p % C::TNE][p / C::TNE] = acc[(h * P + p) % C::TN][(h * P + p) / C::TN];
#pragma unroll
                for (int sender = 0; sender < C::KS - 1; ++sender)
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const v4i v = *reinterpret_cast<const v4i *>(xlane + (((h * (C::KS - 1) + sender) * P + p) * 4 + q) * QUAD_BYTES);
#pragma unroll
                            for (int e = 0; e < 4; ++e) mine[p % C::TNE][p / C::TNE][4 * q + e] += v[e];
                        }
            }
        }
        __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
        __builtin_amdgcn_s_barrier();                                // the exchange area is free for the epilogue
        finish<C, C::TNE, C::TME, STORE, DUMP, ZP>(mine, scv, zwv, lds, wave_all, wave, lane, sub0, fin_nw0, fin_mw0, M, N, s_a, d,
                                                 zp, wsum, y, acc_out, ws, splits, split, pid, total);
    } else {
        load_scales<C::TN, ZP>(scv, zwv, s_w, wsum, fin_nw0, N, lane);
        finish<C, C::TN, C::TM, STORE, DUMP, ZP>(acc, scv, zwv, lds, wave_all, wave, lane, 0, fin_nw0, fin_mw0, M, N, s_a, d, zp,
                                               wsum, y, acc_out, ws, splits, split, pid, total);
    }
}

// 0 = choose the tile shape per problem; 1..8 = force one (testing and tuning)
static std::atomic<int> g_forced_tile{0};
static std::atomic<int> g_tile_map{0};
static std::atomic<int> g_prefill{0};     // 0 = where the six-bit kernel pays, 1 = wherever it can run, 2 = never, 128 / 256 = as 1, with that tile
void set_gemm_tile(int tile) { g_forced_tile.store(tile, std::memory_order_relaxed); }
void set_linear_prefill(int mode) { g_prefill.store(mode, std::memory_order_relaxed); }
void set_gemm_map(int mode) { g_tile_map.store(mode, std::memory_order_relaxed); }
int forced_gemm_tile() { return g_forced_tile.load(std::memory_order_relaxed); }

template <class C, int STORE, bool DUMP, bool ZP>
static hipError_t launch_inst(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                              const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                              hipStream_t s, int32_t *ws = nullptr, int splits = 1)
{
    auto kern = linear_mfma_kernel<C, STORE, DUMP, ZP>;
    const DeviceInfo *info;
    hipError_t e0 = device_info(&info);          // sets every instantiation's LDS attribute on the device's first use
    if (e0 != hipSuccess) return e0;
    int64_t tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    if (tiles_m * tiles_n * splits > 0x7fffffff) return hipErrorInvalidValue;
    kern<<<dim3((unsigned)(tiles_m * tiles_n * splits)), dim3(C::THREADS), C::LDS_BYTES, s>>>(
        xq, wq, (int)M, (int)N, (int)k_tiles(K), (int)tiles_m, (int)tiles_n, s_a, s_w, d, zp, wsum, y, acc, ws, splits, g_tile_map.load(std::memory_order_relaxed));
    return hipGetLastError();
}

template <class C>
static hipError_t launch_cfg(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                             const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                             hipStream_t s, int32_t *ws = nullptr, int splits = 1)
{
#define FPTQ_GEMM_INST(S, D) return wsum ? launch_inst<C, S, D, true>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s, ws, splits) \
                                         : launch_inst<C, S, D, false>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s, ws, splits)
    if (acc) FPTQ_GEMM_INST(ANY_ALIGNMENT, true);
    switch (store_kind(M, N)) {
    case CACHED: FPTQ_GEMM_INST(CACHED, false);
    case STREAMED: FPTQ_GEMM_INST(STREAMED, false);
    default: FPTQ_GEMM_INST(ANY_ALIGNMENT, false);
    }
#undef FPTQ_GEMM_INST
}

// ---- tile shapes (all with 4 waves per K group).  The 256 x 256 tile has the best operand reuse and wins for long
// K; 256 x 128 with two workgroups per CU hides prologue and epilogue and fills partial rounds, and wins elsewhere;
// the 192- and one-workgroup 128-row shapes are kept for shapes neither fits; the K-group shapes serve problems with
// at most one workgroup per CU.
typedef GemmCfg<2, 2, 4, 4, 4> T256x256;           // waves of 128 x 128
typedef GemmCfg<2, 2, 3, 4, 4> T192x256;           // BN = 192: waves of 96 (n) x 128 (m)
typedef GemmCfg<2, 2, 4, 2, 4> T256x128;           // BM = 128: waves of 128 (n) x 64 (m)
typedef GemmCfg<2, 2, 4, 2, 3, 2> T256x128o2;      // the same tile, two workgroups per CU
typedef GemmCfg<2, 2, 2, 2, 3, 1, 2> T128x128k2;   // 128 x 128 alone on a CU, two K groups
typedef GemmCfg<2, 2, 4, 2, 3, 1, 2> T256x128k2;   // 256 x 128 alone on a CU, two K groups
typedef GemmCfg<1, 1, 2, 2, 4, 1, 4> T64x64k4;     // small tiles for problems with few of the larger ones, four K groups:
typedef GemmCfg<2, 1, 2, 2, 3, 1, 4> T128x64k4;    // 64 x 64 with one wave per group, 128 (N) x 64 (M) with two
// split K over workgroups, for problems whose 64 x 64 tiles cover at most half of the CUs
typedef GemmCfg<1, 1, 2, 2, 4, 1, 4, true> T64x64k4split;

// ---- the library's own scratch area, for callers that cannot allocate a workspace: device memory that lives as
// long as the process, one copy per GPU.  Its name is a host-side handle only; the device address is looked up once
// per device (gemm_device_init) and that pointer is what kernels and every other host-side use get.  Sized for the
// split-K exchange on a device of up to 256 CUs: one 64 x 64 INT32 partial tile per workgroup, at most one workgroup
// per CU, plus the counters.  The arrival counters at its start are zero when the code object is loaded and every
// launch leaves them zero (the last workgroup of a tile clears its counter); the partial tiles behind them are
// always written before they are read, so calls in sequence need nothing cleared in between.
constexpr int64_t SCRATCH_BYTES = (int64_t)256 * T64x64k4split::ACC_REGS * 64 * 4 + 4096;
static __device__ __align__(256) int32_t scratch[SCRATCH_BYTES / 4];

template <class C, int STORE, bool DUMP, bool ZP>
static hipError_t set_lds_attribute()
{
    return hipFuncSetAttribute((const void *)linear_mfma_kernel<C, STORE, DUMP, ZP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               C::LDS_BYTES);
}

template <class... Cs>
static hipError_t set_lds_attributes()
{
    hipError_t e = hipSuccess;
    auto one = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    (void)one;
    ((one(set_lds_attribute<Cs, ANY_ALIGNMENT, true, false>()), one(set_lds_attribute<Cs, ANY_ALIGNMENT, true, true>()),
      one(set_lds_attribute<Cs, ANY_ALIGNMENT, false, false>()), one(set_lds_attribute<Cs, ANY_ALIGNMENT, false, true>()),
      one(set_lds_attribute<Cs, CACHED, false, false>()), one(set_lds_attribute<Cs, CACHED, false, true>()),
      one(set_lds_attribute<Cs, STREAMED, false, false>()), one(set_lds_attribute<Cs, STREAMED, false, true>())),
     ...);
    return e;
}

// Once per device, with that device current: every kernel instantiation gets its dynamic-LDS limit (so no launch
// has to set it later, e.g. under graph capture), and the scratch area's address on this device is looked up.
hipError_t gemm_device_init(DeviceInfo *info)
{
    hipError_t e = set_lds_attributes<T256x256, T192x256, T256x128, T256x128o2, T128x128k2, T256x128k2, T64x64k4, T128x64k4,
                                      T64x64k4split>();
    if (e != hipSuccess) return e;
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    info->scratch = static_cast<int32_t *>(ptr);
    info->scratch_bytes = SCRATCH_BYTES;
    return hipSuccess;
}

// Number of K ranges: as many as keep the workgroup count within the CUs, at most MAX_SPLITS, at least 16 K tiles
// (four per K group) each, none empty.  The exchange of partials pays from K = 6144 on (measured on N = 1024,
// M = 256: K = 4096 takes 8.0 us unsplit and 8.6 split, K = 6144 9.8 and 9.0, K = 14336 16.6 and 11.4, K = 28672
// 28.3 and 16.7).
static int64_t split_tiles(int64_t M, int64_t N) { return ((N + T64x64k4split::BN - 1) / T64x64k4split::BN) * ((M + T64x64k4split::BM - 1) / T64x64k4split::BM); }
static int split_count(int64_t M, int64_t N, int64_t K, int cus)
{
    const int64_t tiles = split_tiles(M, N), kt = k_tiles(K);
    if (tiles > cus / 2 || tiles > SPLIT_COUNTERS || K > 131071 || kt < 48) return 1;
    int64_t sp = cus / tiles;
    if (sp > kt / 16) sp = kt / 16;
    if (sp > MAX_SPLITS) sp = MAX_SPLITS;
    if (sp < 2) return 1;
    const int64_t per = (kt + sp - 1) / sp;
    return (int)((kt + per - 1) / per);
}

int64_t linear_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    const int sp = split_count(M, N, K, device_cus_or_default());
    if (sp < 2) return 0;
    const int64_t tiles = split_tiles(M, N);
    return (SPLIT_COUNTERS + sp * tiles * T64x64k4split::ACC_REGS * (T64x64k4split::WAVES * 64)) * 4;
}

hipError_t launch_linear_mfma_ws(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                                 const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                                 int32_t *ws, int64_t ws_bytes, hipStream_t s)
{
    const int sp = split_count(M, N, K, device_cus_or_default());
    if (sp < 2 || !ws || ws_bytes < linear_workspace_bytes(M, N, K) || (wsum && K > 65535) || forced_gemm_tile() != 0)
        return launch_linear_mfma(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    return launch_cfg<T64x64k4split>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s, ws, sp);
}

// Tile shape for a problem: index into the launch table (0 = 256 x 256, 1 = 192 x 256, 2 = 256 x 128, 3 = 256 x 128 with
// two workgroups per CU, 4 = 128 x 128 and 5 = 256 x 128 with two K groups, 6 = 64 x 64 and 7 = 128 x 64 with four).
static int choose_tile(int64_t M, int64_t N, int64_t K, int cus, double *us = nullptr)
{
    const int forced = forced_gemm_tile();
    if (forced > 0) return forced - 1;
    // Estimated time in microseconds, fitted to measurements on uniform random operands on MI355X (the clock is
    // power-limited there, so a K tile costs about the same time whatever the MFMA utilisation):
    // one-workgroup-per-CU shapes run ceil(tiles / CUs) rounds of (fixed + per-K-tile) each.  With two
    // workgroups per CU the older one is served first, so epilogues overlap the other's main loop and
    // a partial last round of r * 2 CUs tiles costs about 0.5 + 0.15 r of a full one instead of 1; a partial
    // only round with more tiles than CUs runs at the pace of the CUs that hold two (0.88 of a full round
    // measured at r = 0.6).  At most one 256 x 128 tile per CU: the two-K-group variant, whose K tiles go
    // faster the fewer CUs are busy (0.67 us at 256 tiles, 0.55 at 160: the power limit again).
    auto tiles = [&](int64_t bn, int64_t bm) { return (double)(((N + bn - 1) / bn) * ((M + bm - 1) / bm)); };
    const double kt = (double)k_tiles(K), CUS = (double)cus;
    const double t21 = tiles(256, 128), x = t21 / (2 * CUS), frac = x - floor(x);
    const double rounds_o2 = x < 1.0 ? 0.7 + 0.3 * x : floor(x) + (frac > 0 ? fmax(frac, 0.5 + 0.15 * frac) : 0.0);
    const double never = 1e30;
    const double cost[5] = {
        ceil(tiles(256, 256) / CUS) * (12.9 + 1.235 * kt),
        ceil(tiles(192, 256) / CUS) * (11.0 + 0.900 * kt),
        t21 > CUS ? ceil(t21 / CUS) * (9.4 + 0.667 * kt) : never,
        // From 64 K tiles on the two large shapes tie in isolated launches, and the tie goes to the 256 x 256 tile: it
        // moves half the operand bytes through L2 and LDS per operation, and in a sustained sequence of launches (the
        // Llama-3-70B layer step, where the clock follows the board's power history) every launch runs 1 to 12 %
        // faster when all of them use it.
        t21 > CUS ? rounds_o2 * (7.8 + 1.304 * kt) * (kt >= 64 ? 1.03 : 1.0) : never,
        t21 <= CUS ? 8.5 + (0.35 + 0.32 * t21 / CUS) * kt : never,
    };
    int pick = 0;
    for (int i = 1; i < 5; ++i)
        if (cost[i] < cost[pick]) pick = i;
    if (us) *us = cost[pick];
    if (pick == 4) pick = 5;       // the launch table: 4 = 128 x 128, 5 = 256 x 128, both with two K groups
    // Problems so small that even 128 x 128 tiles give every CU at most one workgroup take that tile: the
    // kernel time is then one workgroup's walk through K and the small tile walks fastest (17 against 25 us at
    // K = 4096).  A deeper ring does not help there.
    if (tiles(128, 128) <= CUS) {
        pick = 4;
        if (us) *us = 8.0 + (0.30 + 0.08 * tiles(128, 128) / CUS) * kt;
    }
    // Fewer tiles still: the smallest tile shape that still gives every CU at most one workgroup, as four K
    // groups whose waves each hold a whole 64 x 64 block of outputs (half the LDS reads per MFMA of a 32 x 32
    // block).  Measured at K = 4096, N = 4096: 256 tokens 9 us on 64 x 64 tiles against 17 on 128 x 128; 512
    // tokens 12.5 us on 128 x 64 against 18.
    if (tiles(128, 64) <= CUS) pick = 7;
    if (tiles(64, 64) <= CUS) pick = 6;
    if (us && (pick == 6 || pick == 7)) *us = 0.0;     // not estimated: those problems never leave half of the CUs' matrix pipes busy
    return pick;
}

// Whether a problem is faster on the six-bit kernel (fptq_prefill.hip), widening of its activations included, and with how many tokens
// per tile.  Estimated times on uniform random operands, as above, in rounds of one tile of 256 channels per CU: a partial
// last round costs less than a full one (the power it leaves speeds its tiles up), and so does a lone one.  Fitted to 350 shapes of 65 to
// 4096 tokens and checked on 150 others, both with the weights read from HBM, as in a model larger than the last-level cache, and with
// them in that cache, e.g. (us from HBM, the better INT8 shape / 256 / 192 / 128 tokens; in brackets from the cache)
//     2048 x 4096 x 11008    69 /  73 /  65 /  61  (68 / 60 / 59 / 59)     333 x 32000 x 4096   46 / 40 / 36 / 50  (44 / 38 / 33 / 44)
//     1000 x 5120 x 13824    70 /  88 /  67 /  60  (63 / 68 / 59 / 54)     192 x 28672 x 4096   29 / 33 / 31 / 29  (26 / 26 / 24 / 25)
//      700 x 10240 x 8192    52 /  57 /  53 /  45  (49 / 46 / 43 / 43)     512 x 8192 x 8192    34 / 56 / 47 / 39  (33 / 44 / 38 / 32)
// i.e. the tile that leaves the fewest CUs without work, and INT8 where each leaves too many.  Where the smaller tiles occupy less than a share of
// the CUs in a single round (least_share), the estimates spread most and INT8's smaller tiles are closest, so they take 48 K tiles: 562 x 8064 x
// 5376 30 us on INT8 and 37 with 192 tokens, 151 x 19477 x 4472 25 and 33, 1670 x 2560 x 4936 27 and 29 with 128 (weights from HBM).  The 256-token
// tile needs no such limit: refused below four fifths of the CUs, 512 x 23424 x 6016 took 57 us on INT8 instead of 48 (from the cache 54 and 43), 256 x
// 50096 x 2744 36 instead of 30 (33 and 27).  Beyond a round and a half 192 tokens are taken from 25 K tiles on only, where
// they take 2 to 14 % less than what was taken instead on 57 of the 59 shapes of 960 that this concerns, and as long on the other two (2048 x 10240 x
// 8192 91 us against 102 with 256 tokens, 1500 x 14336 x 4096 52 against 62, 3000 x 8192 x 28672 327 against 332; the 256-token tile stays where its
// last round is fuller: 6000 x 5120 x 5120 83 against 88); below that INT8 is as fast.  The margins (wider for few K tiles, where stores and launches
// weigh more than in what the estimates were fitted to, but for the 256-token tile in more than 1.6 rounds from 14 K tiles on: 1732 x 15160 x 3064 55 us
// against 66 on INT8, 1025 x 24520 x 3256 59 against 71) leave 6 of the 960 shapes 5 % or more slower than INT8 with the weights from HBM and 3 from the
// cache, by 12 % at most; the choice takes 0.6 and 0.8 % longer than the best of the four on average (1.2 and 1.6 % without these two rules).
// Tiles of 160 and 96 tokens were within 3 % of the best of the others but on 22 of the first 200 shapes (192 x 28672 x 4096: 26 and 29): not kept.
int prefill_tile(int64_t M, int64_t N, int64_t K)
{
    if (K > 131071 || M > (1 << 24) || N > (1 << 24) || forced_gemm_tile() > 0) return 0;
    const int mode = g_prefill.load(std::memory_order_relaxed);
    if (mode == 2) return 0;
    if (mode > 2) return mode;
    // Half of a tile or more would be padding, and at best it is even: 64 x 57344 x 28672 takes 161 us on INT8 tiles and 159 here, 64 x
    // 57344 x 8192 50 and 52, 64 x 32000 x 16384 58 and 82, 64 x 28672 x 4096 17 and 27.
    if (mode == 0 && M <= 64) return 0;
    const int cus = device_cus_or_default();
    const double kt = (double)k_tiles(K), widen_us = (double)M * (double)K * 1.25 / 5.0e6;
    struct Tile {
        int tokens;
        double call_us, lone, least, tile_us, k_tile_us, least_share;
    };
    static const Tile tiles[] = {{256, 5.0, 0.58, 0.53, 7.5, 0.789, 0.0}, {192, 4.95, 0.54, 0.58, 5.4, 0.649, 0.65}, {128, 5.75, 0.58, 0.69, 3.8, 0.494, 0.76}};
    int tokens = 0;
    double us = 0.0, tile_rounds = 0.0;
    for (const Tile &t : tiles) {
        const int64_t workgroups = prefill_workgroups(M, N, t.tokens);
        const double x = (double)workgroups / (double)cus, part = x - floor(x);
        // A single row of small tiles streams its weights once, from HBM: with few workgroups that is bound by what one CU keeps in flight
        // (96 x 37397 x 17536, 147 workgroups: 92 us against 85 on INT8 tiles; 96 x 57344 x 8192, 224 workgroups: 53 against 53).
        if (t.tokens == 128 && M <= 128 && x < 0.75) continue;
        if (mode == 0 && ((x < t.least_share && kt < 48) || (t.tokens == 192 && x > 1.5 && kt < 25))) continue;
        const double rounds = x < 1.0 ? t.lone + (1.0 - t.lone) * x : floor(x) + (part > 0.0 ? t.least + (1.0 - t.least) * part : 0.0);
        const double est = t.call_us + widen_us + rounds * (t.tile_us + t.k_tile_us * kt);
        if (tokens == 0 || est < us) tokens = t.tokens, us = est, tile_rounds = x;
    }
    if (mode == 1 || tokens == 0) return tokens;
    double int8_us = 0.0;
    choose_tile(M, N, K, cus, &int8_us);
    const bool fitted = kt >= 32 || (kt >= 14 && tokens == 256 && tile_rounds > 1.6);
    return us < (fitted ? 0.94 : 0.85) * int8_us ? tokens : 0;
}

// Limits of the MFMA kernel: the widened accumulator is 256 * acc with |acc| <= 64 K, and one K tile of all rows
// (rows * 64 bytes) must fit a 32-bit buffer descriptor.  Beyond them the simple kernel answers.
static bool mfma_serves(int64_t M, int64_t N, int64_t K, bool zero_point)
{
    return !(K > 131071 || (zero_point && K > 65535) || M > (1 << 24) || N > (1 << 24));
}

template <class C>
static void describe(int64_t M, int64_t N, int splits, LinearPlan *plan)
{
    snprintf(plan->kernel, sizeof plan->kernel, "GemmCfg<%d, %d, %d, %d, %d, %d, %d, %s>", C::WAVES_N, C::WAVES_M, C::TN, C::TM,
             C::STAGES, C::OCC, C::KS, C::SPLIT ? "true" : "false");
    plan->workgroups = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN) * splits;
    plan->threads = C::THREADS;
}

// What launch_linear_mfma / launch_linear_mfma_ws would launch for a shape on the current device (host arithmetic only).
void linear_mfma_plan(int64_t M, int64_t N, int64_t K, bool with_workspace, LinearPlan *plan)
{
    const int cus = device_cus_or_default();
    if (!mfma_serves(M, N, K, false)) {
        snprintf(plan->kernel, sizeof plan->kernel, "linear_ref_kernel");
        plan->workgroups = 0;
        plan->threads = 0;
        return;
    }
    const int sp = with_workspace && forced_gemm_tile() == 0 ? split_count(M, N, K, cus) : 1;
    if (sp >= 2) return describe<T64x64k4split>(M, N, sp, plan);
    switch (choose_tile(M, N, K, cus)) {
    case 1: return describe<T192x256>(M, N, 1, plan);
    case 2: return describe<T256x128>(M, N, 1, plan);
    case 3: return describe<T256x128o2>(M, N, 1, plan);
    case 4: return describe<T128x128k2>(M, N, 1, plan);
    case 5: return describe<T256x128k2>(M, N, 1, plan);
    case 6: return describe<T64x64k4>(M, N, 1, plan);
    case 7: return describe<T128x64k4>(M, N, 1, plan);
    default: return describe<T256x256>(M, N, 1, plan);
    }
}

hipError_t launch_linear_mfma(const uint8_t *xq, const uint8_t *wq, int64_t M, int64_t N, int64_t K, float s_a,
                              const float *s_w, const float *d, int zp, const int32_t *wsum, uint16_t *y, int32_t *acc,
                              hipStream_t s)
{
    if (!mfma_serves(M, N, K, wsum != nullptr)) return launch_linear_ref(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    switch (choose_tile(M, N, K, device_cus_or_default())) {
    case 1: return launch_cfg<T192x256>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 2: return launch_cfg<T256x128>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 3: return launch_cfg<T256x128o2>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 4: return launch_cfg<T128x128k2>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 5: return launch_cfg<T256x128k2>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 6: return launch_cfg<T64x64k4>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    case 7: return launch_cfg<T128x64k4>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    default: return launch_cfg<T256x256>(xq, wq, M, N, K, s_a, s_w, d, zp, wsum, y, acc, s);
    }
}

}  // namespace fptq
