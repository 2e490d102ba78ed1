// FP8 matmul for outputs too small to fill the chip with 256 x 256 tiles
// (decode, batched decode, short prompts, small layers), for gfx950.
// C[m, n] = 2^-(ba + bb) * sum_k A[m, k] * B[n, k], K a multiple of 128.
//
// These products are bound by how fast each compute unit can pull operand
// rows into LDS: it keeps about 128 outstanding 128-byte fills, whatever the
// instruction mix, so the time is (rows of the tile) x K per workgroup times
// the rounds of workgroups.  A workgroup therefore takes a small tile of
// 16 MB x 16 NB outputs, chosen so that the grid is one round (or a few whole
// rounds) of the 256 compute units, and its four waves split k, not the tile:
//  * Every stage copies KC bytes of k of the tile's 16 (MB + NB) rows with
//    global_load_lds_dwordx4 (runs of KC contiguous bytes per row), three
//    stages in LDS, two in flight.  Weight rows that no other workgroup reads
//    carry the non-temporal hint.
//  * KC = 512 (up to 96 rows): wave w multiplies the whole tile over the 128
//    bytes of k at 128 w of each stage.  KC = 256 (up to 192 rows): waves w
//    and w + 2 share a 128-byte slice, each half of the tile's columns.  No
//    fragment is read from LDS twice.
//  * The waves' partial sums are added through LDS in a fixed order, so the
//    result does not depend on timing.
//  * 16-byte chunk c of LDS row r is stored at chunk c ^ (r % 16): the lanes
//    of every ds_read_b128 phase (see fp8lin_gemm.hip) hit distinct banks.
#include "fp8lin_mm.h"

namespace fp8lin {
namespace {

constexpr int kSlBuf = 3;

// Waves 0-3 multiply; with more than 16 rows of A waves 4-7 copy, otherwise
// the multiplying waves copy too (see the main loop).
constexpr bool copy_waves(int mb) { return mb > 1; }
constexpr int stream_threads(int mb) { return copy_waves(mb) ? 512 : 256; }

template <int FA, int FB, int MB, int NB>
__global__ __launch_bounds__(stream_threads(MB)) void gemm_nt_stream(MmArgs p, int tiles_m, int nt) {
    constexpr int kRowsB = 16 * NB, kRows = 16 * (MB + NB);
    constexpr int kKC = MB + NB <= 6 ? 512 : 256;
    constexpr int kStage = kRows * kKC, kCpr = kKC / 16, kRpi = 64 / kCpr;  // chunks per row, rows per copy
    constexpr int kNiw = kRows / kRpi / 4;                                  // copies per wave and stage
    constexpr int kSlots = kKC / 128, kHalves = 4 / kSlots, kNbw = NB / kHalves;
    static_assert(kRows % (4 * kRpi) == 0 && NB % kHalves == 0, "tile split");
    static_assert(kSlBuf * kStage <= 160 * 1024 && kSlots * MB * NB * 1024 <= kSlBuf * kStage, "LDS budget");
    __shared__ __attribute__((aligned(1024))) uint8_t sm[kSlBuf * kStage];
    __shared__ uint32_t wmx[8];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = (int)p.M, N = (int)p.N, K = (int)p.K;
    // consecutive tiles of one XCD share their B rows
    const int x = blockIdx.x & 7, per = gridDim.x >> 3, rem = gridDim.x & 7;
    const int tile = x * per + min(x, rem) + (blockIdx.x >> 3);
    const int m0 = tile % tiles_m * (16 * MB), n0 = tile / tiles_m * kRowsB;

    // copy t of this wave: LDS rows kRpi d .. (d = kNiw w + t), B rows first;
    // rows past the matrix edge read the last row (their outputs are not stored)
    const int lrow = lane / kCpr, lchunk = lane % kCpr;
    uint32_t voff[kNiw];
#pragma unroll
    for (int t = 0; t < kNiw; ++t) {
        const int r = ((w & 3) * kNiw + t) * kRpi + lrow;
        const int src = r < kRowsB ? min(n0 + r, N - 1) - n0 : min(m0 + r - kRowsB, M - 1) - m0;
        voff[t] = (uint32_t)(src * K + ((lchunk ^ (r & 15)) << 4));
    }
    const uint8_t* baseA = p.A + (int64_t)m0 * K;
    const uint8_t* baseB = p.B + (int64_t)n0 * K;
    const uint32_t lds0 = lds_addr(sm);
    const int nst = (K + kKC - 1) / kKC;
    auto issue = [&](int st) {
        const int buf = st % kSlBuf, end = K - st * kKC - 16;  // offset of the row's last chunk
        const bool part = end + 16 < kKC;
#pragma unroll
        for (int t = 0; t < kNiw; ++t) {
            const int d = (w & 3) * kNiw + t;
            const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + buf * kStage + d * 1024);
            uint32_t v = voff[t];
            if (part) {  // chunks past the row end re-read its last one (never multiplied)
                const int c = (lchunk ^ ((d * kRpi + lrow) & 15)) << 4;
                v -= (uint32_t)max(0, c - end);
            }
            if (d * kRpi >= kRowsB) lds_dma16_s(baseA + (int64_t)st * kKC, v, dst);
            else if (nt) lds_dma16_nt(baseB + (int64_t)st * kKC, v, dst);
            else lds_dma16_s(baseB + (int64_t)st * kKC, v, dst);
        }
    };

    const int frow = lane & 15, fg = lane >> 4;
    const int slot = w % kSlots, half = (w & 3) / kSlots;
    const int fo0 = frow * kKC + (((slot * 8 + 2 * fg) ^ frow) << 4);
    const int fo1 = frow * kKC + (((slot * 8 + 2 * fg + 1) ^ frow) << 4);
    v4f acc[MB][kNbw];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < kNbw; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int st) {
        if (st * kKC + slot * 128 >= K) return;
        const uint8_t* sb = sm + (st % kSlBuf) * kStage + half * kNbw * 16 * kKC;
        const uint8_t* sa = sm + (st % kSlBuf) * kStage + kRowsB * kKC;
        v8i bf[kNbw];
#pragma unroll
        for (int j = 0; j < kNbw; ++j) bf[j] = ld_frag(sb + j * 16 * kKC, fo0, fo1);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const v8i af = ld_frag(sa + i * 16 * kKC, fo0, fo1);
#pragma unroll
            for (int j = 0; j < kNbw; ++j) acc[i][j] = mfma16<FB, FA>(bf[j], af, acc[i][j]);
        }
        wait_lgkmcnt0();  // the next barrier frees this buffer
    };
    // wait until stage st has landed, stages up to `issued` being on their way
    auto landed = [&](int st, int issued) {
        if (st < issued) wait_vmcnt<kNiw>();
        else wait_vmcnt<0>();
    };
    if (copy_waves(MB)) {
        // Between barriers st and st + 1 the multiplying waves take stage st
        // and the copying waves issue stage st + 2 into the buffer of stage
        // st - 1 and wait for stage st + 1: an issue that stalls for room
        // among the outstanding fills stalls no multiplication (100 x 12288 x
        // 4096: 23.6 -> 18.0 us, 512 x 8192 x 8192: 93 -> 61 us).
        if (w >= 4) {
            if (nst > 0) issue(0);
            if (nst > 1) issue(1);
            landed(0, nst - 1);
            ws_barrier();
            for (int st = 0; st < nst; ++st) {
                if (st + 2 < nst) issue(st + 2);
                landed(st + 1, nst - 1);
                ws_barrier();
            }
        } else {
            ws_barrier();
            for (int st = 0; st < nst; ++st) {
                multiply(st);
                ws_barrier();
            }
        }
    } else {
        // Few MFMAs per stage: copying waves of their own gain nothing and
        // cost 1-5 % of a stream from HBM (16 x 57344 x 8192: 74.8 against
        // 79.1 us).
        if (nst > 0) issue(0);
        if (nst > 1) issue(1);
        for (int st = 0; st < nst; ++st) {
            landed(st, nst - 1);
            ws_barrier();
            // the buffer of stage st - 1, which every wave has finished reading
            if (st + 2 < nst) issue(st + 2);
            multiply(st);
        }
        ws_barrier();
    }
    v4f* red = (v4f*)sm;  // [slot][16-row block][16-column block][lane]
    if (w < 4) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < kNbw; ++j) red[((slot * MB + i) * NB + half * kNbw + j) * 64 + lane] = acc[i][j];
    }
    __syncthreads();
    uint32_t mx = 0;
    const int bb = *p.bb;
    for (int b = w; b < MB * NB; b += stream_threads(MB) / 64) {
        v4f sum = red[b * 64 + lane];
#pragma unroll
        for (int s = 1; s < kSlots; ++s) sum += red[(s * MB * NB + b) * 64 + lane];
        const int64_t m = m0 + b / NB * 16 + frow, n = n0 + b % NB * 16 + fg * 4;
        if (n >= N) continue;
        const int sh = row_shift(p.ba, p.ba_rows, bb, m, M);
        mx = max(mx, p.out_dt == FP8_DT_BF16 ? store4<FP8_DT_BF16>(p.C, N, m, n, M, N, sum, sh)
                                             : store4<FP8_DT_F32>(p.C, N, m, n, M, N, sum, sh));
    }
    if (p.with_amax) {
        const uint32_t wv = wave_max_u32(mx);
        if (lane == 0) wmx[w] = wv;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t b = 0;
#pragma unroll
            for (int v = 0; v < stream_threads(MB) / 64; ++v) b = max(b, wmx[v]);
            fold_amax(canon_amax(b), p.amax, p.bo);
        }
    }
}

template <int FA, int FB, int MB, int NB>
void launch_one(const MmArgs& a, hipStream_t s) {
    const int tm = (int)((a.M + 16 * MB - 1) / (16 * MB)), tn = (int)((a.N + 16 * NB - 1) / (16 * NB));
    hipLaunchKernelGGL((gemm_nt_stream<FA, FB, MB, NB>), dim3((unsigned)(tm * tn)), dim3(stream_threads(MB)), 0, s, a, tm,
                       tm == 1);
}

// Tile shapes (16-row blocks of A and of B) the kernel is built for: those the
// rule below chooses somewhere for 1 to 2048 rows and weights of 128 to 57344.
#define FP8LIN_STREAM_TILES(X)                                                                             \
    X(1, 1) X(1, 2) X(1, 3) X(1, 4) X(1, 5) X(1, 6) X(1, 8) X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(2, 6) X(2, 8)  \
    X(3, 1) X(3, 2) X(3, 3) X(3, 4) X(3, 6) X(3, 8) X(4, 2) X(4, 4) X(4, 6) X(4, 8) X(5, 2) X(5, 4) X(5, 6) \
    X(6, 4) X(6, 6) X(8, 4)

template <int FA, int FB>
void launch_t(int mb, int nb, const MmArgs& a, hipStream_t s) {
#define FP8LIN_STREAM_CASE(MB, NB) \
    if (mb == MB && nb == NB) return launch_one<FA, FB, MB, NB>(a, s);
    FP8LIN_STREAM_TILES(FP8LIN_STREAM_CASE)
#undef FP8LIN_STREAM_CASE
}

}  // namespace

// Estimated time (us) of the product with tiles of 16 MB x 16 NB: a linear fit
// to 40 shapes x 33 tiles on MI355X (M 1-512, weights 512-57344 wide), which
// picks a tile within 1 % of the best measured one on average (14 % at worst,
// on products of 7 us).  The terms: launch; rounds of workgroups (prologue and
// epilogue); bytes the busiest compute unit copies (83 GB/s each); the weight
// read once from memory; barriers per stage; the weight re-read from L2 by
// each row of tiles.
template <int MB, int NB>
static double stream_us(int64_t M, int64_t N, int64_t K) {
    constexpr int kc = MB + NB <= 6 ? 512 : 256, lds = kSlBuf * 16 * (MB + NB) * kc;
    constexpr int occ = 160 * 1024 / lds < 4 ? 160 * 1024 / lds : 4;
    const int64_t tm = (M + 16 * MB - 1) / (16 * MB), tiles = tm * ((N + 16 * NB - 1) / (16 * NB));
    const int64_t per_cu = (tiles + 255) / 256, rounds = (tiles + 256 * occ - 1) / (256 * occ);
    return 2.28 + 1.645 * rounds + 12.1e-6 * (double)(per_cu * 16 * (MB + NB)) * K + 5.17e-8 * (double)N * K +
           2.31e-4 * (double)rounds * K * 512 / kc + 8.75e-9 * (double)tm * N * K;
}

double stream_tile(int64_t M, int64_t N, int64_t K, int* mb, int* nb) {
    double best = 0;
#define FP8LIN_STREAM_COST(MB, NB)                                     \
    if (const double t = stream_us<MB, NB>(M, N, K); best == 0 || t < best) { \
        best = t;                                                      \
        *mb = MB;                                                      \
        *nb = NB;                                                      \
    }
    FP8LIN_STREAM_TILES(FP8LIN_STREAM_COST)
#undef FP8LIN_STREAM_COST
    return best;
}

void launch_gemm_stream(int fa, int fb, int mb, int nb, const MmArgs& a, hipStream_t s) {
    if (fa == FP8_E4M3 && fb == FP8_E4M3) launch_t<FP8_E4M3, FP8_E4M3>(mb, nb, a, s);
    else if (fa == FP8_E5M2 && fb == FP8_E4M3) launch_t<FP8_E5M2, FP8_E4M3>(mb, nb, a, s);
    else launch_t<FP8_E4M3, FP8_E5M2>(mb, nb, a, s);
}

}  // namespace fp8lin
