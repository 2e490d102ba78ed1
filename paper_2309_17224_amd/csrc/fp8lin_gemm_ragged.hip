// FP8 matmul for contraction lengths that are not a multiple of 128 (the
// grad-weight product over an odd number of tokens, odd layer widths), or of
// 2^22 and more, for gfx950.  C[m, n] = 2^-(ba + bb) * sum_k A[m, k] * B[n, k].
//
// The rows of both operands are dense, so with K not a multiple of 16 they
// start at any byte address: the direct global -> LDS copies of the aligned
// kernels cannot be used.  Here each thread loads its 16-byte chunks into
// registers at the row's own alignment (gfx950 global memory takes unaligned
// 16-byte loads), one k-step ahead, and writes them to LDS rows of 128 bytes,
// 16-byte chunks XOR-swizzled as in the aligned kernels.  The last k-step's
// bytes past the row end are zero in LDS, so they add nothing.  The k order
// inside the sums is that of the 256 x 256 kernel with a zero-padded K.
#include "fp8lin_mm.h"

namespace fp8lin {
namespace {

constexpr int kRk = 128;  // bytes of k per step

// Bytes [k, k + 16) of a row of K bytes, zero from K on; reads only bytes of
// the row.  With K >= 16 one load ending at the row's end, moved down.
__device__ __forceinline__ uint4 ld16_tail(const uint8_t* row, int64_t k, int64_t K) {
    if (K < 16) {  // one or two loads that overlap: sixteen guarded bytes took 1.7 us
        if (k > 0) return make_uint4(0u, 0u, 0u, 0u);
        if (K >= 8) {
            const u32x2_any lo = *(const u32x2_any*)row, hi = *(const u32x2_any*)(row + K - 8);
            const uint64_t h = (hi.x | ((uint64_t)hi.y << 32)) >> 8 >> (8 * (15 - K));
            return make_uint4(lo.x, lo.y, (uint32_t)h, (uint32_t)(h >> 32));
        }
        if (K >= 4) {
            const uint32_t lo = *(const u32_any*)row, hi = *(const u32_any*)(row + K - 4);
            return make_uint4(lo, hi >> 8 >> (8 * (7 - K)), 0u, 0u);
        }
        const uint32_t b0 = row[0], b1 = row[min((int64_t)1, K - 1)], b2 = row[K - 1];
        return make_uint4(b0 | (K > 1 ? b1 << 8 : 0u) | (K > 2 ? b2 << 16 : 0u), 0u, 0u, 0u);
    }
    const int64_t at = min(k, K - 16);
    const int sh = (int)min(k - at, (int64_t)16) * 8;  // bits to drop
    return shr128(ld16_any(row + at), sh);
}

// One BM x BN output tile per workgroup, WT x WT per wave.
template <int FA, int FB, int BM, int BN, int WT>
__global__ __launch_bounds__((BM / WT) * (BN / WT) * 64) void gemm_nt_ragged(MmArgs p, int tiles_m, int tiles_n) {
    constexpr int kNt = (BM / WT) * (BN / WT) * 64, kWaves = kNt / 64;
    constexpr int kRows = BM + BN, kStage = kRows * kRk;
    constexpr int kRpi = kNt / 8;            // rows per load of the workgroup (8 lanes a row)
    constexpr int kNc = kRows / kRpi;        // loads per thread and step
    constexpr int kB = WT / 16;              // 16-row blocks of a wave's sub-tile
    static_assert(kRows % kRpi == 0 && BM % kRpi == 0, "loader rows");
    // epilogue staging: 32 output rows of a wave at a time
    constexpr int kEpRow = WT * 4 + 16, kEpWave = 32 * kEpRow;
    constexpr int kSmem = 2 * kStage > kWaves * kEpWave ? 2 * kStage : kWaves * kEpWave;
    __shared__ __attribute__((aligned(128))) uint8_t smem[kSmem];
    __shared__ uint32_t wmx[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int tm, tn;
    tile_of(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    const int64_t M = p.M, N = p.N, K = p.K;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

    // loader: chunk tid % 8 of rows tid / 8 + i kRpi of the tile (A rows, then
    // B rows); rows past the matrix edge read the last row (not stored)
    const int lc = tid & 7, lr = tid >> 3;
    const uint8_t* row[kNc];
    uint32_t dst[kNc];
#pragma unroll
    for (int i = 0; i < kNc; ++i) {
        const int r = lr + i * kRpi;
        row[i] = i * kRpi < BM ? p.A + min(m0 + r, M - 1) * K : p.B + min(n0 + r - BM, N - 1) * K;
        dst[i] = r * kRk + ((lc ^ chunk_swz(r)) << 4);
    }
    const int nk = (int)((K + kRk - 1) / kRk);
    uint4 rg[kNc];
    auto load = [&](int kt) {
        const int64_t k = (int64_t)kt * kRk + lc * 16;
        if ((int64_t)(kt + 1) * kRk <= K) {
#pragma unroll
            for (int i = 0; i < kNc; ++i) rg[i] = ld16_any(row[i] + k);
        } else if (K % 16 == 0) {  // whole chunks, nothing to shift (1024 x 8 x 64: 4.6 us with)
#pragma unroll
            for (int i = 0; i < kNc; ++i) {
                const uint4 v = ld16_any(row[i] + min(k, K - 16));
                rg[i] = k < K ? v : make_uint4(0u, 0u, 0u, 0u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kNc; ++i) rg[i] = ld16_tail(row[i], k, K);
        }
    };
    auto store = [&](int kt) {
        uint8_t* d = smem + (kt & 1) * kStage;
#pragma unroll
        for (int i = 0; i < kNc; ++i) *(uint4*)(d + dst[i]) = rg[i];
    };

    const int wr0 = (w / (BN / WT)) * WT, wc0 = (w % (BN / WT)) * WT;
    const int frow = lane & 15, fg = lane >> 4;
    const int fo0 = frow * kRk + (((2 * fg) ^ chunk_swz(frow)) << 4);
    const int fo1 = frow * kRk + (((2 * fg + 1) ^ chunk_swz(frow)) << 4);
    v4f acc[kB][kB];
#pragma unroll
    for (int i = 0; i < kB; ++i)
#pragma unroll
        for (int j = 0; j < kB; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    if (nk > 0) {
        load(0);
        store(0);
        if (nk > 1) load(1);
    }
    wait_lgkmcnt0();
    ws_barrier();
    // step kt: write step kt + 1 (loaded during step kt - 1) into the other
    // stage, which every wave finished reading before the last barrier, issue
    // the loads of step kt + 2, multiply step kt
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) {
            store(kt + 1);
            if (kt + 2 < nk) load(kt + 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t* sa = smem + (kt & 1) * kStage + wr0 * kRk;
        const uint8_t* sb = smem + (kt & 1) * kStage + (BM + wc0) * kRk;
        v8i af[kB], bf[kB];
#pragma unroll
        for (int i = 0; i < kB; ++i) af[i] = ld_frag(sa + i * 16 * kRk, fo0, fo1);
#pragma unroll
        for (int j = 0; j < kB; ++j) bf[j] = ld_frag(sb + j * 16 * kRk, fo0, fo1);
#pragma unroll
        for (int i = 0; i < kB; ++i)
#pragma unroll
            for (int j = 0; j < kB; ++j) acc[i][j] = mfma16<FB, FA>(bf[j], af[i], acc[i][j]);
        wait_lgkmcnt0();
        ws_barrier();
    }

    // Epilogue: unscale, round once, stage 32 rows of the wave at a time in
    // LDS (its own region) and store 16-byte pieces of whole row runs.
    uint8_t* ep = smem + w * kEpWave;
    const int bb = *p.bb;
    uint32_t mx = 0;
#pragma unroll
    for (int i2 = 0; i2 < WT / 32; ++i2) {
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            const int i = 2 * i2 + ii;
            const int sh = row_shift(p.ba, p.ba_rows, bb, m0 + wr0 + i * 16 + frow, M);
#pragma unroll
            for (int j = 0; j < kB; ++j) {
                const v4f a = acc[i][j];
                const float y[4] = {ldexpf(a[0], sh), ldexpf(a[1], sh), ldexpf(a[2], sh), ldexpf(a[3], sh)};
                uint8_t* e = ep + (ii * 16 + frow) * kEpRow;
                if (p.out_dt == FP8_DT_BF16) {
                    const uint32_t lo = pack_bf16x2(y[0], y[1]), hi = pack_bf16x2(y[2], y[3]);
                    mx = max(mx, max(max(lo & 0x7FFFu, (lo >> 16) & 0x7FFFu), max(hi & 0x7FFFu, (hi >> 16) & 0x7FFFu)) << 16);
                    *(uint2*)(e + (j * 16 + 4 * fg) * 2) = make_uint2(lo, hi);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) mx = max(mx, __float_as_uint(y[v]) & 0x7FFFFFFFu);
                    *(float4*)(e + (j * 16 + 4 * fg) * 4) = make_float4(y[0], y[1], y[2], y[3]);
                }
            }
        }
        wait_lgkmcnt0();
        const int esz = p.out_dt == FP8_DT_BF16 ? 2 : 4;
        const int lpr = WT * esz / 16, per = 16 / esz;  // lanes per row, elements per lane
        for (int r = lane / lpr; r < 32; r += 64 / lpr) {
            const int cc = lane % lpr;
            const uint4 v = *(const uint4*)(ep + r * kEpRow + cc * 16);
            const int64_t m = m0 + wr0 + i2 * 32 + r, n = n0 + wc0 + cc * per;
            if (m >= M || n >= N) continue;
            uint8_t* o = (uint8_t*)p.C + (m * N + n) * esz;
            if (n + per <= N) {
                st_stream(o, v);
            } else {
                const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                for (int e = 0; e < per && n + e < N; ++e) {
                    if (esz == 2) ((uint16_t*)o)[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
                    else ((uint32_t*)o)[e] = wv[e];
                }
            }
        }
        wait_lgkmcnt0();  // the staging rows may be overwritten
    }
    if (p.with_amax) {  // rows and columns past the edge are copies of real ones
        const uint32_t wv = wave_max_u32(mx);
        if (lane == 0) wmx[w] = wv;
        __syncthreads();
        if (tid == 0) {
            uint32_t b = 0;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) b = max(b, wmx[v]);
            fold_amax(canon_amax(b), p.amax, p.bo);
        }
    }
}

// Tiles of 256 x 128 from 128 of them on, else of 64 x 64.
bool big_tiles(int64_t M, int64_t N) { return ((M + 255) / 256) * ((N + 127) / 128) >= 128; }

template <int FA, int FB, int BM, int BN, int WT>
void launch_tiles(const MmArgs& a, hipStream_t s) {
    const int tm = (int)((a.M + BM - 1) / BM), tn = (int)((a.N + BN - 1) / BN);
    hipLaunchKernelGGL((gemm_nt_ragged<FA, FB, BM, BN, WT>), dim3((unsigned)(tm * tn)), dim3((BM / WT) * (BN / WT) * 64), 0, s,
                       a, tm, tn);
}

template <int FA, int FB>
void launch_t(const MmArgs& a, hipStream_t s) {
    if (big_tiles(a.M, a.N)) launch_tiles<FA, FB, 256, 128, 64>(a, s);
    else launch_tiles<FA, FB, 64, 64, 32>(a, s);
}

}  // namespace

int64_t ragged_workgroups(int64_t M, int64_t N) {
    return big_tiles(M, N) ? ((M + 255) / 256) * ((N + 127) / 128) : ((M + 63) / 64) * ((N + 63) / 64);
}

void launch_gemm_ragged(int fa, int fb, const MmArgs& a, hipStream_t s) {
    if (fa == FP8_E4M3 && fb == FP8_E4M3) launch_t<FP8_E4M3, FP8_E4M3>(a, s);
    else if (fa == FP8_E5M2 && fb == FP8_E4M3) launch_t<FP8_E5M2, FP8_E4M3>(a, s);
    else launch_t<FP8_E4M3, FP8_E5M2>(a, s);  // the products of the ABI: E4 x E4, E5 x E4, E4 x E5
}

}  // namespace fp8lin
