// FP8 x FP8 -> fp32 matmul with the unscale 2^-(b_a + b_b) fused into the
// epilogue (Sec. 2 and 2.2; Eq. 2), for gfx950 matrix cores.
//
// C[m, n] = 2^-(ba + bb) * sum_k A[m, k] * B[n, k]   ("NT": both operands
// are contiguous along the contraction index).  The forward pass, the
// grad-input and the grad-weight products of the linear layer are all of
// this form once the casts have written the transposed copies they need.
//
// Main kernel (K a multiple of 128, 16-byte aligned operands):
//  * 256 x 256 output tile per workgroup of 8 waves, two per SIMD (wave w
//    runs on SIMD w % 4).  Each wave owns a 64 x 128 sub-tile = 4 x 8 blocks
//    of v_mfma_f32_16x16x128_f8f6f4; the two waves of a SIMD own the two
//    halves of one 128 x 128 quadrant.
//  * K advances 128 bytes at a time; both operand tiles (256 rows x 128 B)
//    go HBM/L2 -> LDS with global_load_lds_dwordx4 (no VGPR staging): A into
//    two stages, B into three (all 160 KiB of LDS).
//  * The copies are slow to issue (the L1 holds only so many outstanding
//    fills): group 0 copies the A tiles and group 1 the B tiles, each in its
//    own load phase, so both load phases share the cost.
//  * The two waves of a SIMD alternate between an MFMA phase and a load
//    phase, the phases separated by workgroup barriers: while one issues its
//    32 MFMAs of step k, the other reads all its fragments of its next step
//    into registers and issues the copies of its operand for a later step.
//    The matrix core of each SIMD is fed by one wave at a time, and the
//    cost of issuing vector-memory and LDS instructions falls on the wave
//    that is not feeding it (see the main loop).
//  * LDS rows are 128 B; the 16-byte chunk index is XOR-swizzled with the row
//    (chunk ^ chunk_swz(row), below) by choosing which global chunk each lane
//    fetches.  The LDS has 64 four-byte banks (16 groups of 16 bytes) and
//    serves a ds_read_b128 in four phases of 16 lanes: lane bit 5 and the
//    parity of lane bits 2, 3 and 4 select the phase (measured on gfx950 with
//    a sweep of address patterns; lanes 0-15 are NOT one phase).  The swizzle
//    gives the 16 lanes of every phase of a fragment read distinct bank groups.
//  * A fragment of the 16x16x128 MFMA is 32 bytes per lane: row (lane % 16),
//    32 consecutive k of group (lane / 16).  The matrix core pairs the same
//    register bytes of both operands, so any k order that is the same for
//    both operands gives the same dot products.
//  * The MFMA gets the B fragment as its first operand, so each lane's four
//    accumulators are four consecutive n of one m: the epilogue writes 8 B
//    (bf16) or 16 B (fp32) per lane.
//  * Workgroup -> tile mapping: workgroups are dealt round-robin to the 8
//    XCDs; the remap gives each XCD a contiguous range of tiles, walked in
//    groups of 8 tile-rows, so tiles sharing operand panels meet in the same
//    L2.
// Outputs too small for these tiles, decode among them: fp8lin_gemm_stream.hip.
// K not a multiple of 128, or K >= 2^22: fp8lin_gemm_ragged.hip.
#include <algorithm>

#include "fp8lin_mm.h"

namespace fp8lin {
namespace {

// ------------------------------------------------------------ main kernel
constexpr int kBM = 256, kBN = 256, kBK = 128;
constexpr int kMainThreads = 512;      // 8 waves: two groups of four
constexpr int kTileBytes = kBM * kBK;  // one operand tile, 32 KiB

__device__ __forceinline__ int bq_used(const int32_t* pred) { return clamp_bias(*pred); }

// Epilogue staging rows (bytes): 32 output rows of a wave per pass; the
// codes of the fused quantise (256 x 256 bytes) follow the bf16 staging area.
constexpr int kEpRowBf16 = 128 * 2 + 16, kEpRowF32 = 128 * 4 + 16;
constexpr int kEpBf16Bytes = 8 * 32 * kEpRowBf16, kEpF32Bytes = 8 * 32 * kEpRowF32;
constexpr int kCodesOff = kEpBf16Bytes;
constexpr int kEpBytes = kCodesOff + kBM * kBN > kEpF32Bytes ? kCodesOff + kBM * kBN : kEpF32Bytes;
// Main loop: two A stages and three B stages (B tiles are copied two steps
// ahead, see gemm_tile); the epilogue reuses the space, and the workgroup's
// amax words sit in its last 64 bytes, past every epilogue staging area.
constexpr int kSmemBytes = 2 * kTileBytes + 3 * kBN * kBK;
constexpr int kWmxOff = kSmemBytes - 64;
static_assert(kEpBytes <= kWmxOff && kSmemBytes <= 160 * 1024, "LDS budget");
static_assert(kCodesOff % 16 == 0, "codes staging alignment");

// Output codes of the fused quantise (QF >= 0, bf16 output only): Y8 [M, N]
// and optionally Y8T [N, M] in format QF, cast with a predicted bias; the
// tile maxima and the prediction used go to a workspace for the exact-bias
// check (see launch_gemm_nt_quantise).
struct QuantOut {
    const int32_t* pred;  // predicted bias (device)
    int32_t* used;        // out: the clamped prediction the codes were cast with
    uint32_t* parts;      // out: per-workgroup largest |Y| pattern (bf16 bits)
    uint8_t* y8;
    int64_t ldy8;
    uint8_t* y8t;  // may be null
    int64_t ldy8t;
};

// One output tile of 256 rows x TN columns (TN = 64..256; each wave owns 64
// rows x TN/2 columns), tile number bid of nb in this workgroup's share of the
// launch, over columns [col0, col0 + tiles_n TN) of C.  The last workgroup of
// the launch takes the bias when bo.ws is set.
template <int FA, int FB, int OUT_DT, bool AMAX, int QF, int TN>
__device__ __forceinline__ void gemm_tile(
    uint8_t* __restrict__ smem, int bid, int nb, const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
    const int32_t* __restrict__ ba_p, const int32_t* __restrict__ bb_p, void* __restrict__ C, int M, int N, int K,
    int tiles_m, int tiles_n, int col0, uint32_t* __restrict__ amax_out, const QuantOut& qo,
    const BiasOut& bo, int ba_rows) {
    static_assert(QF < 0 || OUT_DT == FP8_DT_BF16, "fused quantise is for bf16 outputs");
    static_assert(QF < 0 || TN == 256, "fused quantise stages whole 256 x 256 tiles");
    static_assert(TN % 64 == 0 && TN >= 64 && TN <= 256, "tile width");
    constexpr int kNbw = TN / 32;                  // 16-column blocks per wave, B copies per loader wave
    constexpr int kBStage = TN * kBK;              // one B tile in LDS
    constexpr int kNf = 4 + kNbw;                  // fragment pieces a wave reads per step
    constexpr int kNc = 8 + kNbw;                  // copies a loader wave issues per stage

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // group (0: waves 0-3, 1: waves 4-7) and quadrant; wave-uniform
    const int g = __builtin_amdgcn_readfirstlane(w >> 2), sq = __builtin_amdgcn_readfirstlane(w & 3);
    int tm, tn;
    tile_of(bid, nb, tiles_m, tiles_n, tm, tn);
    const int m0 = tm * kBM, n0 = col0 + tn * TN;

    // Loader (group 0): wave sq fills rows [64 sq, 64 sq + 64) of the A tile
    // and [TN/4 sq, TN/4 (sq + 1)) of the B tile, 8 rows per copy (voff[0..7]
    // for A, voff[8..] for B); lane -> row r = (first row) + 8 i + lane / 8 and
    // physical chunk lane % 8, which holds logical chunk (lane % 8) ^
    // chunk_swz(r).  Rows past the matrix edge re-read the last row (their
    // outputs are not stored).  Offsets are relative to the tile's first row,
    // so they fit 32 bits for K < 2^22.
    const int lrow = lane >> 3;
    uint32_t voff[kNc];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = sq * 64 + i * 8 + lrow;
        voff[i] = (uint32_t)((min(m0 + r, M - 1) - m0) * K + ((lane & 7) ^ chunk_swz(r)) * 16);
    }
#pragma unroll
    for (int i = 0; i < kNbw; ++i) {
        const int r = sq * (TN / 4) + i * 8 + lrow;
        voff[8 + i] = (uint32_t)((min(n0 + r, N - 1) - n0) * K + ((lane & 7) ^ chunk_swz(r)) * 16);
    }
    const uint8_t* baseA = A + (int64_t)m0 * K;
    const uint8_t* baseB = B + (int64_t)n0 * K;
    // LDS addresses of this wave's first loader rows (wave-uniform); copy d
    // < 8 fills A row group d, copy d >= 8 B row group d - 8.
    // LDS: A stages 0 and 1 at s * kTileBytes, B stages 0, 1 and 2 after them.
    const uint32_t lds_a = __builtin_amdgcn_readfirstlane(lds_addr(smem) + sq * 64 * kBK);
    const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_addr(smem) + 2 * kTileBytes + sq * (TN / 4) * kBK);
    auto dma = [&](int d, int stage, int k0) {  // stage: of A for d < 8, of B for d >= 8
        lds_dma16_s((d >= 8 ? baseB : baseA) + k0, voff[d],
                    d >= 8 ? lds_b + (d - 8) * 8 * kBK + stage * kBStage : lds_a + d * 8 * kBK + stage * kTileBytes);
    };

    // this wave's sub-tile: rows [wr0, wr0 + 64), columns [wc0, wc0 + TN/2) of the tile
    const int wr0 = (sq >> 1) * 128 + g * 64, wc0 = (sq & 1) * (TN / 2);
    const int frow = lane & 15, fg = lane >> 4;
    // byte offsets (within a 16-row block) of this lane's two fragment pieces
    const int fo0 = frow * kBK + (((2 * fg) ^ chunk_swz(frow)) << 4);
    const int fo1 = frow * kBK + (((2 * fg + 1) ^ chunk_swz(frow)) << 4);

    v4f acc[4][kNbw];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < kNbw; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // Ping-pong pipeline.  Phases are separated by workgroup barriers; in
    // every phase one group issues MFMAs and the other loads:
    //   phase 1:        group 0 loads fragments of step 0
    //   phase 2k + 2:   group 0 MFMAs of step k,   group 1 loads step k
    //   phase 2k + 3:   group 0 loads step k + 1,  group 1 MFMAs of step k
    // A load phase reads all kNf fragment pieces of the wave's next step and
    // waits for them before the barrier.  A tile k sits in A stage k % 2, B
    // tile k in B stage k % 3.  Group 0 copies A tile k + 1 in its load phase
    // of step k (after both groups have read A tile k - 1 from that stage) and
    // waits for the copies at the end of its next MFMA phase.  Group 1 copies
    // B tile k + 2 in its load phase of step k (B tile k - 1 has been read by
    // then) and, before that phase's barrier, waits for B tile k + 1 — issued
    // one load phase earlier — but not for the copies it has just issued.
    // Steps 0 and 1 are copied before phase 1.  Every wave passes 2 nk + 1
    // barriers (group 1 passes one before its first load phase and none after
    // its last MFMA phase), so the groups stay in step.
    const int nk = K / kBK;
    if (nk > 0) {
        if (g == 0) {
#pragma unroll
            for (int d = 0; d < 8; ++d) dma(d, 0, 0);
            if (nk > 1) {
#pragma unroll
                for (int d = 0; d < 8; ++d) dma(d, 1, kBK);
                wait_vmcnt<8>();
            } else {
                wait_vmcnt<0>();
            }
        } else {
#pragma unroll
            for (int d = 8; d < kNc; ++d) dma(d, 0, 0);
            if (nk > 1) {
#pragma unroll
                for (int d = 8; d < kNc; ++d) dma(d, 1, kBK);
                wait_vmcnt<kNbw>();
            } else {
                wait_vmcnt<0>();
            }
        }
        ws_barrier();
        if (g == 1) ws_barrier();
    }
    v8i af[4], bf[kNbw];
    int bs = 0;  // k % 3: the B stage of step k
    for (int kt = 0; kt < nk; ++kt) {
        const uint8_t* sa = smem + (kt & 1) * kTileBytes + wr0 * kBK;
        const uint8_t* sb = smem + 2 * kTileBytes + bs * kBStage + wc0 * kBK;
        if (g == 0 && kt >= 1 && kt + 1 < nk) {
            // A tile of step kt + 1, the copies spread over the fragment reads
            const int st = (kt + 1) & 1, k1 = (kt + 1) * kBK;
#pragma unroll
            for (int q = 0; q < kNf; ++q) {
                if (q < 4) af[q] = ld_frag(sa + q * 16 * kBK, fo0, fo1);
                else bf[q - 4] = ld_frag(sb + (q - 4) * 16 * kBK, fo0, fo1);
                if (q < 8) dma(q, st, k1);
            }
#pragma unroll
            for (int d = kNf; d < 8; ++d) dma(d, st, k1);
        } else if (g == 1 && kt + 2 < nk) {
            // B tile of step kt + 2 into the stage B tile kt - 1 used
            const int st = bs == 0 ? 2 : bs - 1, k2 = (kt + 2) * kBK;
#pragma unroll
            for (int q = 0; q < kNf; ++q) {
                if (q < 4) af[q] = ld_frag(sa + q * 16 * kBK, fo0, fo1);
                else bf[q - 4] = ld_frag(sb + (q - 4) * 16 * kBK, fo0, fo1);
                if (q < kNbw) dma(8 + q, st, k2);
            }
        } else {
#pragma unroll
            for (int q = 0; q < kNf; ++q) {
                if (q < 4) af[q] = ld_frag(sa + q * 16 * kBK, fo0, fo1);
                else bf[q - 4] = ld_frag(sb + (q - 4) * 16 * kBK, fo0, fo1);
            }
        }
        if (g == 1) {  // B tile kt + 1 has landed (the copies just issued need not have)
            if (kt + 2 < nk) wait_vmcnt<kNbw>();
            else wait_vmcnt<0>();
        }
        bs = bs == 2 ? 0 : bs + 1;
        wait_lgkmcnt0();
        ws_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < kNbw; ++j) {
                acc[i][j] = mfma16<FB, FA>(bf[j], af[i], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        if (g == 0) {
            wait_vmcnt<0>();
            ws_barrier();
        } else if (kt + 1 < nk) {
            ws_barrier();
        }
    }

    // Epilogue: y = 2^-(ba + bb) acc (exact ldexp), rounded once to the output
    // type, staged through LDS 32 rows at a time per wave so that every global
    // store writes 16-byte pieces of whole 256-byte (bf16) or 512-byte (fp32)
    // row runs.  Staging reads map one LDS read phase (lane bit 5 and the
    // parity of lane bits 2..4) to one row, so they are free of bank conflicts.
    // The last barrier of the main loop follows every read of the operand
    // tiles, so group 0 stages and stores its outputs while group 1 issues its
    // last MFMAs.
    int shr[4];  // unscale exponent of this lane's rows wr0 + 16 i + frow
#pragma unroll
    for (int i = 0; i < 4; ++i) shr[i] = row_shift(ba_p, ba_rows, *bb_p, (int64_t)m0 + wr0 + i * 16 + frow, M);
    const int prow = 2 * (lane >> 5) + (((lane >> 2) ^ (lane >> 3) ^ (lane >> 4)) & 1);
    uint32_t mx = 0;
    if (OUT_DT == FP8_DT_BF16) {
        uint8_t* ep = smem + w * 32 * kEpRowBf16;
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        u16x2 m2 = {0, 0};
        // Fused quantise: the codes of the tile, row-major, after the staging
        // rows (row r = 256 bytes; 16-byte chunk c stored at chunk c ^ (r % 16)).
        uint8_t* cs = smem + kCodesOff;
        int bq = 0;
        uint32_t codes[4][8];
        if (QF >= 0) bq = clamp_bias(*qo.pred);
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2) {
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int i = 2 * i2 + ii;
#pragma unroll
                for (int j = 0; j < kNbw; ++j) {
                    const uint32_t lo = pack_bf16x2(ldexpf(acc[i][j][0], shr[i]), ldexpf(acc[i][j][1], shr[i]));
                    const uint32_t hi = pack_bf16x2(ldexpf(acc[i][j][2], shr[i]), ldexpf(acc[i][j][3], shr[i]));
                    if (AMAX || QF >= 0) {
                        m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2, lo & 0x7FFF7FFFu));
                        m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2, hi & 0x7FFF7FFFu));
                    }
                    if (QF >= 0) {
                        uint32_t c4 = cast4_bf16<QF < 0 ? 0 : QF>(lo, hi, bq);
                        if (__builtin_expect(any_nan_bf16(lo, hi), 0)) {
                            const uint32_t hs[4] = {lo & 0xFFFFu, lo >> 16, hi & 0xFFFFu, hi >> 16};
                            c4 = nan_patch<QF < 0 ? 0 : QF>(c4, hs);
                        }
                        codes[i][j] = c4;
                        const int r = wr0 + i * 16 + frow, col = wc0 + j * 16 + 4 * fg;
                        *(uint32_t*)(cs + r * 256 + ((((col >> 4) ^ r) & 15) << 4) + (col & 15)) = c4;
                    }
                    *(uint2*)(ep + (ii * 16 + frow) * kEpRowBf16 + (j * 16 + 4 * fg) * 2) = make_uint2(lo, hi);
                }
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int row = 4 * t + prow, c16 = lane & 15;
                const uint4 v = *(const uint4*)(ep + row * kEpRowBf16 + c16 * 16);
                const int64_t m = m0 + wr0 + i2 * 32 + row, n = n0 + wc0 + c16 * 8;
                if (m < M && c16 < TN / 16) {
                    uint16_t* p = (uint16_t*)C + m * N + n;
                    if (n + 8 <= N) {
                        st_stream(p, v);
                    } else {
                        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                        for (int e = 0; e < 8 && n + e < N; ++e) p[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        }
        mx = (uint32_t)max(m2.x, m2.y) << 16;
        if (QF >= 0) {
            // Y8 rows from the staged codes: 4096 chunks of 16 bytes, 8 per thread.
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const int idx = threadIdx.x + h * kMainThreads, r = idx >> 4, c = idx & 15;
                const uint4 v = *(const uint4*)(cs + r * 256 + (((c ^ r) & 15) << 4));
                const int64_t m = m0 + r, n = n0 + c * 16;
                if (m < M && n < N) {
                    uint8_t* p = qo.y8 + m * qo.ldy8 + n;
                    if (n + 16 <= N) {
                        st16_any(p, v);
                    } else {
                        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                        for (int e = 0; e < 16 && n + e < N; ++e) p[e] = (uint8_t)(wv[e >> 2] >> (8 * (e & 3)));
                    }
                }
            }
            if (qo.y8t) {
                // Y8T: restage the codes column-major (column c = 256 bytes of
                // rows; chunk q of column c stored at chunk q ^ (c % 16)).
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int r = wr0 + i * 16 + frow, col0 = wc0 + j * 16 + 4 * fg;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int c = col0 + e;
                            cs[c * 256 + ((((r >> 4) ^ c) & 15) << 4) + (r & 15)] = (uint8_t)(codes[i][j] >> (8 * e));
                        }
                    }
                __syncthreads();
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    const int idx = threadIdx.x + h * kMainThreads, c = idx >> 4, q = idx & 15;
                    const uint4 v = *(const uint4*)(cs + c * 256 + (((q ^ c) & 15) << 4));
                    const int64_t n = n0 + c, m = m0 + q * 16;
                    if (n < N && m < M) {
                        uint8_t* p = qo.y8t + n * qo.ldy8t + m;
                        if (m + 16 <= M) {
                            st16_any(p, v);
                        } else {
                            const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                            for (int e = 0; e < 16 && m + e < M; ++e) p[e] = (uint8_t)(wv[e >> 2] >> (8 * (e & 3)));
                        }
                    }
                }
            }
        }
    } else {
        uint8_t* ep = smem + w * 32 * kEpRowF32;
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2) {
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int i = 2 * i2 + ii;
#pragma unroll
                for (int j = 0; j < kNbw; ++j) {
                    float y[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        y[v] = ldexpf(acc[i][j][v], shr[i]);
                        if (AMAX) mx = max(mx, __float_as_uint(y[v]) & 0x7FFFFFFFu);
                    }
                    *(float4*)(ep + (ii * 16 + frow) * kEpRowF32 + (j * 16 + 4 * fg) * 4) =
                        make_float4(y[0], y[1], y[2], y[3]);
                }
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int row = 2 * t + (lane >> 5), c32 = lane & 31;
                const float4 v = *(const float4*)(ep + row * kEpRowF32 + c32 * 16);
                const int64_t m = m0 + wr0 + i2 * 32 + row, n = n0 + wc0 + c32 * 4;
                if (m < M && c32 < TN / 8) {
                    float* p = (float*)C + m * N + n;
                    if (n + 4 <= N) {
                        st_stream(p, make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)));
                    } else {
                        const float fv[4] = {v.x, v.y, v.z, v.w};
                        for (int e = 0; e < 4 && n + e < N; ++e) p[e] = fv[e];
                    }
                }
            }
        }
    }
    if (AMAX || QF >= 0) {
        // The workgroup's largest |Y| pattern: one global atomic per workgroup
        // (the waves of all resident workgroups finish together, and atomics
        // on one word from every wave would queue behind each other).  Rows
        // and columns past the edge computed clamped copies of real ones, so
        // including them cannot change the maximum.
        uint32_t* wmx = (uint32_t*)(smem + kWmxOff);
        const uint32_t wv = wave_max_u32(mx);
        if (lane == 0) wmx[w] = wv;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t b = 0;
#pragma unroll
            for (int v = 0; v < kMainThreads / 64; ++v) b = max(b, wmx[v]);
            if (AMAX) fold_amax(canon_amax(b), amax_out, bo);
            if (QF >= 0) {  // bf16 magnitude pattern
                qo.parts[blockIdx.x] = b >> 16;
                if (blockIdx.x == 0) *qo.used = bq_used(qo.pred);
            }
        }
    }
}

// The 256-row kernel.  Workgroups below g1 take 256 x 256 tiles (tiles_m x
// tiles_n of them); with TN2 > 0 the rest take tiles TN2 wide over the
// columns after them (tiles_m x tiles_n2), a last round of narrower tiles
// instead of a partial round of full ones (see narrow_split).  g1 is a whole
// number of rounds of 8 workgroups per XCD, so both parts keep their XCD
// layout.
template <int FA, int FB, int OUT_DT, bool AMAX, int QF = -1, int TN2 = 0>
__global__ __launch_bounds__(kMainThreads) void gemm_nt_256(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, const int32_t* __restrict__ ba_p,
    const int32_t* __restrict__ bb_p, void* __restrict__ C, int M, int N, int K, int tiles_m,
    int tiles_n, uint32_t* __restrict__ amax_out, QuantOut qo, BiasOut bo, int ba_rows,
    int g1, int tiles_n2) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kSmemBytes];
    const int b = blockIdx.x;
    if (TN2 == 0 || b < g1)
        gemm_tile<FA, FB, OUT_DT, AMAX, QF, 256>(smem, b, TN2 == 0 ? (int)gridDim.x : g1, A, B, ba_p, bb_p, C, M, N,
                                                 K, tiles_m, tiles_n, 0, amax_out, qo, bo, ba_rows);
    else
        gemm_tile<FA, FB, OUT_DT, AMAX, -1, (TN2 > 0 ? TN2 : 256)>(smem, b - g1, (int)gridDim.x - g1, A, B, ba_p,
                                                                   bb_p, C, M, N, K, tiles_m, tiles_n2, tiles_n * kBN,
                                                                   amax_out, qo, bo, ba_rows);
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// Workgroups of the 256-row kernel that run at once (one per CU of gfx950).
constexpr int kRound = 256;

// The bias of a launch whose workgroups folded their maxima into bo.ws[0].
__global__ void bias_finish_kernel(uint32_t* amax_out, BiasOut bo) {
    if (threadIdx.x != 0) return;
    const uint32_t a = bo.ws[0];
    bo.ws[0] = 0u;
    uint32_t fl;
    *bo.bias = bias_of_fmt(bo.fmt, a, bo.margin, &fl);
    if (amax_out) *amax_out = a;
    if (bo.flags) *bo.flags = fl;
}

// Most workgroups of a small-tile launch that take the bias in the launch
// itself.  Small tiles finish together, and the device performs one atomic on
// a word after another: 9 ns for a fold alone, 18 ns for a fold and a count,
// which a launch of bias_finish_kernel would save from 64 workgroups on (in the
// launch and after it: 128 workgroups 8.4 and 8.0 us, 192 10.8 and 9.1, 256
// 12.0 and 10.0).  But the host takes 3.7 us to launch it, which is what bounds
// small layers called one by one (training step of 1024 x 768 x 768: 73 us, 80
// with two such launches), so only outputs of more tiles than compute units
// take it.  The 256 x 256 tiles are few or finish apart.
constexpr int64_t kFoldInLaunch = 256;

// Columns of 256-wide tiles taken in whole rounds of kRound workgroups, and
// the rest in one round of narrower tiles: with all 256-wide, a last partial
// round costs as much as a full one.  E.g. 4096 x 11008 (16 x 43 tiles):
// two rounds over the first 8192 columns, then 240 tiles 192 wide (0.75 of
// the work each) over the last 2816.  Every output is still computed by one
// workgroup over the whole K in the same order, so the bits do not change.
// ndp: 256-wide tile columns; tw, tn2: width and count of the narrow ones
// (tw = 0: no narrow launch).
void narrow_split(int tiles_m, int tiles_n, int64_t N, int& ndp, int& tw, int& tn2) {
    ndp = tiles_n;
    tw = 0;
    tn2 = 0;
    const int64_t T = (int64_t)tiles_m * tiles_n;
    if (T % kRound == 0 || tiles_m > kRound) return;
    int gcd = kRound, b = tiles_m;
    while (b) {
        const int t = gcd % b;
        gcd = b;
        b = t;
    }
    const int step = kRound / gcd;  // tile columns per whole number of rounds
    const int c = tiles_n / step * step;
    const int64_t nrem = N - (int64_t)c * kBN;
    for (int w : {64, 128, 192}) {
        const int64_t strips = (nrem + w - 1) / w;
        if (tiles_m * strips <= kRound) {
            ndp = c;
            tw = w;
            tn2 = (int)strips;
            return;
        }
    }
}

// Estimated time (us) of gemm_nt_256: a fit to its times at 33 to 2048 rows
// and weights 512 to 57344 wide, on codes of normal data, weights in cache and
// not (4 % off on average).  Per k-step: a part for each round of 256-wide
// tiles; for the round of narrower ones, a part that does not depend on their
// number and one that does; a part that grows as the operand panels of one XCD
// (up to 8 tile rows of A, its eighth of B) outgrow its 4 MB of L2.  Then the
// weight read once, and the output.
double main_us(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles_m = (M + kBM - 1) / kBM, tiles_n = (N + kBN - 1) / kBN;
    int ndp, tw, tn2;
    narrow_split((int)tiles_m, (int)tiles_n, N, ndp, tw, tn2);
    const double part = (double)(tiles_m * tn2) / kRound;
    const double weight = (double)N * (double)K, panels = (double)std::min<int64_t>(M, 8 * kBM) * (double)K + weight / 8;
    const double step = 1.24 * (double)((tiles_m * ndp + kRound - 1) / kRound) +
                        (tw == 64 ? 0.479 + 0.026 * part : tw == 128 ? 0.129 + 0.489 * part : tw == 192 ? 0.171 + 0.564 * part : 0) +
                        0.142 * std::min(1.0, std::max(0.0, (panels * 1e-6 - 3) / 3));
    return 4.554 + (double)(K / kBK) * step + 4.93e-8 * weight + 2.193e-7 * (double)M * (double)N;
}

template <int FA, int FB, int OUT_DT, bool AMAX>
void launch_t(const MmRoute& r, const uint8_t* A, const int32_t* ba, const uint8_t* B, const int32_t* bb, void* C,
              int64_t M, int64_t N, int64_t K, uint32_t* amax, const BiasOut& bo, int ba_rows, hipStream_t s) {
    if (r.kernel == kMmRagged) {
        launch_gemm_ragged(FA, FB, MmArgs{A, B, ba, bb, C, M, N, K, OUT_DT, AMAX, amax, bo, ba_rows}, s);
    } else if (r.kernel == kMmStream) {
        launch_gemm_stream(FA, FB, r.mb, r.nb, MmArgs{A, B, ba, bb, C, M, N, K, OUT_DT, AMAX, amax, bo, ba_rows}, s);
    } else {
        const int tiles_m = (int)((M + kBM - 1) / kBM), tiles_n = (int)((N + kBN - 1) / kBN);
        int ndp, tw, tn2;
        narrow_split(tiles_m, tiles_n, N, ndp, tw, tn2);
        const int g1 = tiles_m * ndp, grid = g1 + tiles_m * tn2;
#define FP8LIN_GEMM256(TW)                                                                                         \
    hipLaunchKernelGGL((gemm_nt_256<FA, FB, OUT_DT, AMAX, -1, TW>), dim3(grid), dim3(kMainThreads), 0, s, A, B, ba, \
                       bb, C, (int)M, (int)N, (int)K, tiles_m, ndp, amax, QuantOut{}, bo, ba_rows, g1, tn2)
        if (tw == 64) FP8LIN_GEMM256(64);
        else if (tw == 128) FP8LIN_GEMM256(128);
        else if (tw == 192) FP8LIN_GEMM256(192);
        else FP8LIN_GEMM256(0);
#undef FP8LIN_GEMM256
    }
}

// with_amax: epilogue amax (into *amax, or folded into bo.ws).
template <int FA, int FB>
void dispatch_out(const MmRoute& r, const uint8_t* A, const int32_t* ba, const uint8_t* B, const int32_t* bb, void* C,
                  int out_dt, int64_t M, int64_t N, int64_t K, bool with_amax, uint32_t* amax,
                  const BiasOut& bo, int ba_rows, hipStream_t s) {
    if (out_dt == FP8_DT_BF16) {
        if (with_amax) launch_t<FA, FB, FP8_DT_BF16, true>(r, A, ba, B, bb, C, M, N, K, amax, bo, ba_rows, s);
        else launch_t<FA, FB, FP8_DT_BF16, false>(r, A, ba, B, bb, C, M, N, K, amax, bo, ba_rows, s);
    } else {
        if (with_amax) launch_t<FA, FB, FP8_DT_F32, true>(r, A, ba, B, bb, C, M, N, K, amax, bo, ba_rows, s);
        else launch_t<FA, FB, FP8_DT_F32, false>(r, A, ba, B, bb, C, M, N, K, amax, bo, ba_rows, s);
    }
}

void dispatch_fmts(const MmRoute& r, const uint8_t* A, int fa, const int32_t* ba, const uint8_t* B, int fb, const int32_t* bb,
                   void* C, int out_dt, int64_t M, int64_t N, int64_t K, bool with_amax, uint32_t* amax,
                   const BiasOut& bo, int ba_rows, hipStream_t s) {
    if (fa == FP8_E4M3 && fb == FP8_E4M3)
        dispatch_out<FP8_E4M3, FP8_E4M3>(r, A, ba, B, bb, C, out_dt, M, N, K, with_amax, amax, bo, ba_rows, s);
    else if (fa == FP8_E5M2 && fb == FP8_E4M3)
        dispatch_out<FP8_E5M2, FP8_E4M3>(r, A, ba, B, bb, C, out_dt, M, N, K, with_amax, amax, bo, ba_rows, s);
    else  // the ABI's products: E4 x E4, E5 x E4, E4 x E5
        dispatch_out<FP8_E4M3, FP8_E5M2>(r, A, ba, B, bb, C, out_dt, M, N, K, with_amax, amax, bo, ba_rows, s);
}

template <int FA, int FB, int QF>
void launch_fused_t(const uint8_t* A, const int32_t* ba, const uint8_t* B, const int32_t* bb, void* C,
                    int64_t M, int64_t N, int64_t K, const QuantOut& qo, hipStream_t s) {
    const int tiles_m = (int)((M + kBM - 1) / kBM), tiles_n = (int)((N + kBN - 1) / kBN);
    hipLaunchKernelGGL((gemm_nt_256<FA, FB, FP8_DT_BF16, false, QF>), dim3(tiles_m * tiles_n), dim3(kMainThreads), 0,
                       s, A, B, ba, bb, C, (int)M, (int)N, (int)K, tiles_m, tiles_n, nullptr, qo, BiasOut{}, 0,
                       tiles_m * tiles_n, 0);
}

template <int FA, int FB>
void fused_fmt(int qfmt, const uint8_t* A, const int32_t* ba, const uint8_t* B, const int32_t* bb, void* C,
               int64_t M, int64_t N, int64_t K, const QuantOut& qo, hipStream_t s) {
    switch (qfmt) {
        case FP8_E4M3: launch_fused_t<FA, FB, FP8_E4M3>(A, ba, B, bb, C, M, N, K, qo, s); break;
        case FP8_E5M2: launch_fused_t<FA, FB, FP8_E5M2>(A, ba, B, bb, C, M, N, K, qo, s); break;
        case FP8_E4_A: launch_fused_t<FA, FB, FP8_E4_A>(A, ba, B, bb, C, M, N, K, qo, s); break;
        default: launch_fused_t<FA, FB, FP8_E5_A>(A, ba, B, bb, C, M, N, K, qo, s); break;
    }
}

}  // namespace

// The LDS-staged kernels need K a multiple of 128 and 32-bit offsets within a
// tile.  The small tiles (fp8lin_gemm_stream.hip) take up to 32 rows always,
// and beyond that where they are estimated to be faster: of 700 measured
// products of 33 to 2048 rows the choice is slower than gemm_nt_256 on five,
// by 1 to 4 % but for 160 x 15360 x 5120 (36.3 against 32.7 us), and 0.6 % off
// the best on average: 512 x 8192 x 8192 45.5 against 48.3 us, 1024 x 768 x 768
// 6.0 against 7.8, 64 x 4096 x 11008 16.8 against 55.8; 1024 x 4096 x 4096 27.8
// against 26.4 and 100 x 22016 x 4096 32.8 against 26.1, so those go there.
MmRoute mm_route(int64_t M, int64_t N, int64_t K, bool with_amax) {
    if (K % kBK != 0 || K >= (1 << 22)) return {kMmRagged, 0, 0};
    MmRoute r{kMmStream, 0, 0};
    const double us = stream_tile(M, N, K, with_amax, &r.mb, &r.nb);
    if (M <= 32) return r;
    const int64_t tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN);
    if (tiles <= 16 * kRound && us < main_us(M, N, K)) return r;
    return {kMm256, 0, 0};
}

int64_t gemm_quantise_ws_words(int64_t M, int64_t N) {
    const int64_t tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN);
    const int64_t q = quantise_ws_words(M, N);
    return 1 + tiles > q ? 1 + tiles : q;
}

int32_t launch_gemm_nt_quantise(const uint8_t* A, int fa, const int32_t* ba, const uint8_t* B, int fb,
                                const int32_t* bb, void* C, int64_t M, int64_t N, int64_t K, int qfmt,
                                int32_t margin, const int32_t* pred, int32_t* bias, uint32_t* amax_bits,
                                uint32_t* flags, uint8_t* y8, int64_t ldy8, uint8_t* y8t, int64_t ldy8t,
                                uint32_t* ws, hipStream_t s) {
    // The kernel of the plain product, whose bits the fused call promises.
    // Where small tiles win there, they win the whole call with the separate
    // quantise too: 125 such products of 33 to 2048 rows took 0.3 to 0.81 of
    // the fused call's time with a prediction that holds or misses (1024 x 768
    // x 768 18.5 -> 12.9 us, 512 x 8192 x 8192 72.3 -> 51.9).
    const MmRoute route = mm_route(M, N, K, false);
    const bool fused = pred && route.kernel == kMm256 && (fa == FP8_E4M3 || fa == FP8_E5M2) && fb == FP8_E4M3;
    if (!fused) {  // matmul, then the quantise of its output (same bits, more passes)
        const int32_t st = launch_gemm_nt(A, fa, ba, B, fb, bb, C, FP8_DT_BF16, M, N, K, nullptr, s, 0, &route);
        if (st != FP8_OK) return st;
        return launch_quantise(C, FP8_DT_BF16, M, N, N, qfmt, margin, pred, bias, amax_bits, flags, y8, ldy8, y8t,
                               ldy8t, ws, s);
    }
    QuantOut qo;
    qo.pred = pred;
    qo.used = (int32_t*)ws;
    qo.parts = ws + 1;
    qo.y8 = y8;
    qo.ldy8 = ldy8;
    qo.y8t = y8t;
    qo.ldy8t = ldy8t;
    if (fa == FP8_E4M3)
        fused_fmt<FP8_E4M3, FP8_E4M3>(qfmt, A, ba, B, bb, C, M, N, K, qo, s);
    else
        fused_fmt<FP8_E5M2, FP8_E4M3>(qfmt, A, ba, B, bb, C, M, N, K, qo, s);
    const int tiles = (int)(((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN));
    const int32_t st = hip_status();
    if (st != FP8_OK) return st;
    return launch_quant_check(C, FP8_DT_BF16, M, N, N, qfmt, margin, ws + 1, tiles, (int32_t*)ws, bias, amax_bits,
                              flags, y8, ldy8, y8t, ldy8t, s);
}

int32_t launch_fill_u32(uint32_t* p, uint32_t v, hipStream_t s) {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, p, v);
    return hip_status();
}

int32_t launch_gemm_nt(const uint8_t* A, int fa, const int32_t* ba, const uint8_t* B, int fb,
                       const int32_t* bb, void* C, int out_dt, int64_t M, int64_t N, int64_t K,
                       uint32_t* amax_bits, hipStream_t s, int ba_rows, const MmRoute* route) {
    if (amax_bits) hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, amax_bits, 0u);
    dispatch_fmts(route ? *route : mm_route(M, N, K, amax_bits != nullptr), A, fa, ba, B, fb, bb, C, out_dt, M, N, K,
                  amax_bits != nullptr, amax_bits, BiasOut{}, ba_rows, s);
    return hip_status();
}

int32_t launch_gemm_nt_bias(const uint8_t* A, int fa, const int32_t* ba, const uint8_t* B, int fb,
                            const int32_t* bb, void* C, int out_dt, int64_t M, int64_t N, int64_t K, int bfmt,
                            int32_t margin, int32_t* bias, uint32_t* amax_bits, uint32_t* flags, uint32_t* ws,
                            hipStream_t s, int ba_rows, const MmRoute* route) {
    const MmRoute r = route ? *route : mm_route(M, N, K, true);
    const BiasOut bo{bias, flags, ws, bfmt, margin};
    const int64_t wgs = r.kernel == kMmStream ? stream_workgroups(M, N, r.mb, r.nb)
                        : r.kernel == kMmRagged ? ragged_workgroups(M, N) : 0;
    if (wgs <= kFoldInLaunch) {
        dispatch_fmts(r, A, fa, ba, B, fb, bb, C, out_dt, M, N, K, true, amax_bits, bo, ba_rows, s);
    } else {
        dispatch_fmts(r, A, fa, ba, B, fb, bb, C, out_dt, M, N, K, true, ws, BiasOut{}, ba_rows, s);
        hipLaunchKernelGGL(bias_finish_kernel, dim3(1), dim3(64), 0, s, amax_bits, bo);
    }
    return hip_status();
}

}  // namespace fp8lin
