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
//    fragment is read from LDS twice.  KC = 128 (256 rows): the waves take
//    quarters of the tile, and k is not split (512 x 8192 x 8192: 67 us in
//    256-row tiles, 61 in 8 x 4, 48 in 8 x 8).
//  * The partial sums are added through LDS in a fixed order, so the
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
constexpr int stream_kc(int mb, int nb) { return mb + nb <= 6 ? 512 : mb + nb <= 12 ? 256 : 128; }

template <int FA, int FB, int MB, int NB>
__global__ __launch_bounds__(stream_threads(MB)) void gemm_nt_stream(MmArgs p, int tiles_m, int nt) {
    constexpr int kRowsB = 16 * NB, kRows = 16 * (MB + NB);
    constexpr int kKC = stream_kc(MB, NB);
    constexpr int kStage = kRows * kKC, kCpr = kKC / 16, kRpi = 64 / kCpr;  // chunks per row, rows per copy
    constexpr int kNiw = kRows / kRpi / 4;                                  // copies per wave and stage
    constexpr int kSlots = kKC / 128;
    constexpr int kWn = kSlots == 4 ? 1 : 2, kWm = kSlots == 1 ? 2 : 1;  // waves over the tile's columns, rows
    constexpr int kNbw = NB / kWn, kMbw = MB / kWm;
    static_assert(kRows % (4 * kRpi) == 0 && NB % kWn == 0 && MB % kWm == 0, "tile split");
    static_assert(kSlBuf * kStage <= 160 * 1024 && (kSlots == 1 || kSlots * MB * NB * 1024 <= kSlBuf * kStage), "LDS budget");
    __shared__ __attribute__((aligned(1024))) uint8_t sm[kSlBuf * kStage];
    __shared__ uint32_t wmx[8];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = (int)p.M, N = (int)p.N, K = (int)p.K;
    // consecutive tiles of one XCD share their B rows
    const int x = blockIdx.x & 7, per = gridDim.x >> 3, rem = gridDim.x & 7;
    const int tile = x * per + min(x, rem) + (blockIdx.x >> 3);
    int tm = tile % tiles_m, tn = tile / tiles_m;
    if (kSlots == 1) tile_of(blockIdx.x, gridDim.x, tiles_m, (N + kRowsB - 1) / kRowsB, tm, tn);
    const int m0 = tm * (16 * MB), n0 = tn * kRowsB;
    // 16-byte chunk c of LDS row r is stored at chunk c ^ swz(r)
    auto swz = [](int r) { return kKC == 128 ? chunk_swz(r) : r & 15; };

    // copy t of this wave: LDS rows kRpi d .. (d = kNiw w + t), B rows first;
    // rows past the matrix edge read the last row (their outputs are not stored)
    const int lrow = lane / kCpr, lchunk = lane % kCpr;
    uint32_t voff[kNiw];
#pragma unroll
    for (int t = 0; t < kNiw; ++t) {
        const int r = ((w & 3) * kNiw + t) * kRpi + lrow;
        const int src = r < kRowsB ? min(n0 + r, N - 1) - n0 : min(m0 + r - kRowsB, M - 1) - m0;
        voff[t] = (uint32_t)(src * K + ((lchunk ^ swz(r)) << 4));
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
                const int c = (lchunk ^ swz(d * kRpi + lrow)) << 4;
                v -= (uint32_t)max(0, c - end);
            }
            if (d * kRpi >= kRowsB) lds_dma16_s(baseA + (int64_t)st * kKC, v, dst);
            else if (nt) lds_dma16_nt(baseB + (int64_t)st * kKC, v, dst);
            else lds_dma16_s(baseB + (int64_t)st * kKC, v, dst);
        }
    };

    const int frow = lane & 15, fg = lane >> 4;
    const int slot = w % kSlots, part = (w & 3) / kSlots;
    const int nb0 = part % kWn * kNbw, mb0 = part / kWn * kMbw;  // this wave's blocks of the tile
    const int fo0 = frow * kKC + (((slot * 8 + 2 * fg) ^ swz(frow)) << 4);
    const int fo1 = frow * kKC + (((slot * 8 + 2 * fg + 1) ^ swz(frow)) << 4);
    v4f acc[kMbw][kNbw];
#pragma unroll
    for (int i = 0; i < kMbw; ++i)
#pragma unroll
        for (int j = 0; j < kNbw; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int st) {
        if (st * kKC + slot * 128 >= K) return;
        const uint8_t* sb = sm + (st % kSlBuf) * kStage + nb0 * 16 * kKC;
        const uint8_t* sa = sm + (st % kSlBuf) * kStage + (kRowsB + mb0 * 16) * kKC;
        v8i bf[kNbw];
#pragma unroll
        for (int j = 0; j < kNbw; ++j) bf[j] = ld_frag(sb + j * 16 * kKC, fo0, fo1);
#pragma unroll
        for (int i = 0; i < kMbw; ++i) {
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
    uint32_t mx = 0;
    const int bb = *p.bb;
    auto put = [&](int mb, int nb, v4f sum) {
        const int64_t m = m0 + mb * 16 + frow, n = n0 + nb * 16 + fg * 4;
        if (n >= N) return;
        const int sh = row_shift(p.ba, p.ba_rows, bb, m, M);
        mx = max(mx, p.out_dt == FP8_DT_BF16 ? store4<FP8_DT_BF16>(p.C, N, m, n, M, N, sum, sh)
                                             : store4<FP8_DT_F32>(p.C, N, m, n, M, N, sum, sh));
    };
    if (kSlots == 1) {
        if (w < 4) {
#pragma unroll
            for (int i = 0; i < kMbw; ++i)
#pragma unroll
                for (int j = 0; j < kNbw; ++j) put(mb0 + i, nb0 + j, acc[i][j]);
        }
    } else {
        v4f* red = (v4f*)sm;  // [slot][16-row block][16-column block][lane]
        if (w < 4) {
#pragma unroll
            for (int i = 0; i < kMbw; ++i)
#pragma unroll
                for (int j = 0; j < kNbw; ++j) red[((slot * MB + i) * NB + nb0 + j) * 64 + lane] = acc[i][j];
        }
        __syncthreads();
        for (int b = w; b < MB * NB; b += stream_threads(MB) / 64) {
            v4f sum = red[b * 64 + lane];
#pragma unroll
            for (int s = 1; s < kSlots; ++s) sum += red[(s * MB * NB + b) * 64 + lane];
            put(b / NB, b % NB, sum);
        }
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
// rule below chooses somewhere for 1 to 2048 rows and weights of 128 to 57344
// ((1, 4), (4, 2) and (8, 4) only for calls that take the amax).
#define FP8LIN_STREAM_TILES(X)                                                                             \
    X(1, 1) X(1, 2) X(1, 3) X(1, 4) X(1, 5) X(1, 6) X(1, 8) X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(2, 6) X(2, 8)  \
    X(3, 1) X(3, 2) X(3, 3) X(3, 4) X(3, 6) X(3, 8) X(4, 2) X(4, 4) X(4, 6) X(4, 8) X(5, 2) X(5, 4) X(5, 6) \
    X(6, 4) X(6, 6) X(8, 4) X(8, 8) X(10, 6)

template <int FA, int FB>
void launch_t(int mb, int nb, const MmArgs& a, hipStream_t s) {
#define FP8LIN_STREAM_CASE(MB, NB) \
    if (mb == MB && nb == NB) return launch_one<FA, FB, MB, NB>(a, s);
    FP8LIN_STREAM_TILES(FP8LIN_STREAM_CASE)
#undef FP8LIN_STREAM_CASE
}

}  // namespace

// Estimated time (us) of the product with tiles of 16 MB x 16 NB: linear fits
// to 220 shapes x 31 tiles on MI355X (M 1-1500, weights 512-57344 wide), one
// for each kind of tile, which pick a tile within 0.4 % of the best measured
// one on average (12 % at worst, on products of 7 us).
struct StreamFit {
    double launch, round,     // once; per round of workgroups (prologue, epilogue)
        copy, copy_alone,     // MB copied by the busiest compute unit; shared out over its resident workgroups
        stage, mfma,          // its k-bytes of one tile row; its 16 x 16 blocks times k
        weight, weight_part,  // 100 MB of weight; scaled by how much of the last round is empty
        weight_l2, out;       // GB of weight over all rows of tiles; 1e7 outputs
};
constexpr StreamFit kFitDecode{3.479, 0, 2.252, 10.7, 1.913, 0, 0, 6.091, 0, 49.961};   // MB = 1, M <= 16
constexpr StreamFit kFitRows16{1.9, 0.945, 3.85, 16.168, 1.062, 0, 0, 2.467, 0, 13.651};  // MB = 1, M > 16
constexpr StreamFit kFitWide16{2.642, 0.877, 8.195, 0, 9.952, 0, 7.805, 0, 0, 10.343};    // MB = 1, KC = 256
constexpr StreamFit kFit512{2.092, 1.166, 0, 11.704, 2.084, 29.093, 2.814, 1.35, 0, 18.941};
constexpr StreamFit kFit256{2.158, 1.72, 0, 8.853, 5.36, 23.636, 3.739, 1.877, 0, 12.579};
constexpr StreamFit kFit128{2.519, 5.459, 0, 6.509, 0, 35.324, 0, 6.546, 1.301, 6.557};

int64_t stream_workgroups(int64_t M, int64_t N, int mb, int nb) {
    return ((M + 16 * mb - 1) / (16 * mb)) * ((N + 16 * nb - 1) / (16 * nb));
}

// A decode's weight streams through as many workgroups as it takes, and the
// rounds cost nothing but the bytes where each copies for some microseconds.
// With rows as short as these each round past the first adds about this much
// (1 x 57344 x 128: 9.8 us in the 1792 workgroups of 32 columns, 6.7 in 448 of
// 128; 1 x 22016 x 768 7.1 and 5.4 in 230 of 96).
constexpr int64_t kShortK = 2304;
constexpr double kShortRoundUs = 1.0;

template <int MB, int NB>
static double stream_us(int64_t M, int64_t N, int64_t K) {
    constexpr int kc = stream_kc(MB, NB), lds = kSlBuf * 16 * (MB + NB) * kc;
    constexpr int occ = 160 * 1024 / lds < 4 ? 160 * 1024 / lds : 4;
    const StreamFit& f = kc == 128 ? kFit128 : kc == 256 ? (MB == 1 ? kFitWide16 : kFit256)
                         : MB > 1  ? kFit512
                         : M <= 16 ? kFitDecode
                                   : kFitRows16;
    const int64_t tm = (M + 16 * MB - 1) / (16 * MB), tiles = tm * ((N + 16 * NB - 1) / (16 * NB));
    const int64_t rounds = (tiles + 256 * occ - 1) / (256 * occ), per_cu = (tiles + 255) / 256;
    const double cu_k = (double)per_cu * (double)K, mb_copied = cu_k * 16 * (MB + NB) * 1e-6;
    const double weight = (double)N * (double)K * 1e-8;
    const double empty = tiles > 256 * occ ? (double)(rounds * 256 * occ) / (double)tiles : 1.0;
    const double round = &f == &kFitDecode && K <= kShortK ? kShortRoundUs * (double)(rounds - 1) : f.round * (double)rounds;
    return f.launch + round + f.copy * mb_copied + f.copy_alone * mb_copied / (double)(per_cu < occ ? per_cu : occ) +
           f.stage * cu_k * 1e-4 + f.mfma * cu_k * (MB * NB) * 1e-6 + (f.weight + f.weight_part * empty) * weight +
           f.weight_l2 * (double)tm * weight * 0.1 + f.out * (double)M * (double)N * 1e-7;
}

// Every workgroup's fold of its maximum into one word waits for those before
// it, part of which hides behind workgroups that are still multiplying (us).
constexpr double kFoldUs = 0.009;

// The tile with the smallest estimate.  With an epilogue amax, of the tiles
// that sum in the same order (the same KC), so that an output's bits do not
// depend on whether its amax is asked for, the best one with the folds counted
// (256 x 768 x 768 with its amax: 14.4 us in the 768 workgroups that are best
// without, 8.1 in 96; in gemm_nt_256 10.2).
double stream_tile(int64_t M, int64_t N, int64_t K, bool with_amax, int* mb, int* nb) {
    double best = 0;
    int kc = 0;
#define FP8LIN_STREAM_COST(MB, NB)                                                                             \
    if (16 * (MB - 1) < M || MB == 1)                                                                          \
        if (const double t = stream_us<MB, NB>(M, N, K); best == 0 || t < best) {                              \
            best = t;                                                                                          \
            *mb = MB;                                                                                          \
            *nb = NB;                                                                                          \
            kc = stream_kc(MB, NB);                                                                            \
        }
    FP8LIN_STREAM_TILES(FP8LIN_STREAM_COST)
#undef FP8LIN_STREAM_COST
    if (!with_amax) return best;
    double best_fold = 0;
#define FP8LIN_STREAM_COST(MB, NB)                                                                             \
    if ((16 * (MB - 1) < M || MB == 1) && stream_kc(MB, NB) == kc)                                             \
        if (const double t = stream_us<MB, NB>(M, N, K) + kFoldUs * (double)stream_workgroups(M, N, MB, NB);   \
            best_fold == 0 || t < best_fold) {                                                                 \
            best_fold = t;                                                                                     \
            *mb = MB;                                                                                          \
            *nb = NB;                                                                                          \
        }
    FP8LIN_STREAM_TILES(FP8LIN_STREAM_COST)
#undef FP8LIN_STREAM_COST
    return best;
}

bool stream_tile_at(int i, int* mb, int* nb) {
#define FP8LIN_STREAM_ENTRY(MB, NB) {MB, NB},
    static constexpr int tiles[][2] = {FP8LIN_STREAM_TILES(FP8LIN_STREAM_ENTRY)};
#undef FP8LIN_STREAM_ENTRY
    if (i < 0 || i >= (int)(sizeof(tiles) / sizeof(tiles[0]))) return false;
    *mb = tiles[i][0];
    *nb = tiles[i][1];
    return true;
}

void launch_gemm_stream(int fa, int fb, int mb, int nb, const MmArgs& a, hipStream_t s) {
    if (fa == FP8_E4M3 && fb == FP8_E4M3) launch_t<FP8_E4M3, FP8_E4M3>(mb, nb, a, s);
    else if (fa == FP8_E5M2 && fb == FP8_E4M3) launch_t<FP8_E5M2, FP8_E4M3>(mb, nb, a, s);
    else launch_t<FP8_E4M3, FP8_E5M2>(mb, nb, a, s);
}

}  // namespace fp8lin
