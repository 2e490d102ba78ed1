// Per-tensor amax, scaling bias (Sec. 2.3 Eq. 3) and scale-and-cast to FP8
// (Sec. 2.1 Eq. 1) for gfx950.
//
// amax: the absolute maximum is taken as the integer maximum of the
// sign-cleared bit patterns.  For finite values the order of the patterns is
// the order of the magnitudes, NaN patterns sort above infinity, and -0
// clears to 0, so the result is exact and independent of the reduction order.
// Pass 1 reduces to one partial per workgroup (coalesced 16-byte loads, packed
// 16-bit max for bf16); pass 2 (one workgroup) reduces the partials and turns
// the amax into the bias with integer arithmetic.
//
// cast: x * 2^b is formed with v_ldexp_f32, which is exact for every bf16 /
// fp32 x (a power-of-two scale; results below the fp32 normal range are far
// below half the smallest FP8 subnormal and become signed zeros either way),
// clipped to +-max_num with v_med3_f32 (App. A: overflow clips to the
// maximum; infinities included), and converted two at a time by
// v_cvt_pk_fp8_f32 / v_cvt_pk_bf8_f32, which round to nearest even and keep
// subnormals.  The converters encode NaN inputs as 0xFF / 0xFE and overflow
// as NaN or infinity; the clip removes the overflow case and NaN inputs,
// detected with a packed integer test, are re-encoded as 0x7F with their sign.
// The transposed copy goes through a 128 x 128 byte LDS tile so that both
// outputs leave as coalesced stores (whole 128-byte lines for the transpose).
#include <type_traits>

#include "fp8lin_fp8.h"
#include "fp8lin_internal.h"

namespace fp8lin {
namespace {

// Each workgroup reads one contiguous range of 16-byte vectors (a multiple of
// 4 KiB, so ranges start on DRAM-page-friendly boundaries) with eight
// non-temporal loads in flight per lane: a range per workgroup keeps every
// HBM channel streaming through whole pages, which reads measurably faster
// than a grid-stride sweep (about 7 vs 5.5 TB/s on a 2 GiB buffer).
template <int DT>
__global__ __launch_bounds__(kAmaxThreads) void amax_partial_kernel(const void* __restrict__ x,
                                                                   int64_t n,
                                                                   uint32_t* __restrict__ partial) {
    __shared__ uint32_t red[kAmaxThreads / 64];
    constexpr int kL = 8, kSmall = 4;
    uint32_t m = 0;
    constexpr int per = DT == FP8_DT_BF16 ? 8 : 4, esz = 16 / per;
    auto elem = [&](int64_t j) { return DT == FP8_DT_BF16 ? (uint32_t)((const uint16_t*)x)[j] : ((const uint32_t*)x)[j]; };
    constexpr uint32_t kMag = DT == FP8_DT_BF16 ? 0x7FFFu : 0x7FFFFFFFu;
    if (n <= kSmall * kAmaxThreads) {  // one workgroup, elements (100 bf16: 4.3 us by vectors)
        uint32_t e[kSmall];
#pragma unroll
        for (int l = 0; l < kSmall; ++l) e[l] = elem(min((int64_t)threadIdx.x + l * kAmaxThreads, n - 1));
#pragma unroll
        for (int l = 0; l < kSmall; ++l) m = max(m, e[l] & kMag);
        m = block_max(m, red);
        if (threadIdx.x == 0) partial[blockIdx.x] = m;
        return;
    }
    // Whole vectors from the first 16-byte boundary on: unaligned vectors of
    // lines in cache take a quarter longer (2048 x 4096 bf16 one element off:
    // 9.9 us, 6.2 this way).  The few elements before and after them are one
    // per thread of block 0, on their way before the vectors.
    const int64_t head = min(n, (int64_t)((-(uintptr_t)x & 15) / esz));
    const uint4* __restrict__ p = (const uint4*)((const char*)x + head * esz);
    const int64_t nv = (n - head) / per;
    const bool outside = blockIdx.x == 0 && threadIdx.x < n - nv * per;
    uint32_t edge = 0;
    if (blockIdx.x == 0) {
        const int64_t j = outside ? (threadIdx.x < head ? threadIdx.x : threadIdx.x + nv * per) : 0;
        edge = elem(j);
    }
    const int64_t chunk = ((nv + gridDim.x - 1) / gridDim.x + 255) & ~(int64_t)255;
    const int64_t b0 = min(nv, (int64_t)blockIdx.x * chunk), b1 = min(nv, b0 + chunk);
    int64_t i = b0 + threadIdx.x;
    us2 mm = {0, 0};
    auto fold = [&](const uint4& v) {
        if (DT == FP8_DT_BF16) mm = fold_bf16(mm, v);
        else m = fold_f32(m, v);
    };
    for (; i + (kL - 1) * kAmaxThreads < b1; i += kL * kAmaxThreads) {
        uint4 v[kL];
#pragma unroll
        for (int l = 0; l < kL; ++l) v[l] = ld_stream(p + i + l * kAmaxThreads);
        // all kL loads issue before the first use (the scheduler would
        // otherwise start folding the first one and wait for it alone)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int l = 0; l < kL; ++l) fold(v[l]);
    }
    // fewer than kL vectors of this lane left: unconditional loads of
    // in-range vectors (a guarded load compiles to a branch and a wait per
    // load), those past the range replaced by zero, neutral for the maximum
    if (b1 > b0) {
        uint4 v[kL];
#pragma unroll
        for (int l = 0; l < kL; ++l) v[l] = ld_stream(p + min(i + l * kAmaxThreads, b1 - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int l = 0; l < kL; ++l)
            if (i + l * kAmaxThreads >= b1) v[l] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int l = 0; l < kL; ++l) fold(v[l]);
    }
    if (DT == FP8_DT_BF16) m = max((uint32_t)mm.x, (uint32_t)mm.y);
    if (outside) m = max(m, edge & kMag);
    m = block_max(m, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

template <int DT, int FMT>
__global__ __launch_bounds__(kAmaxThreads) void amax_finalize_kernel(
    const uint32_t* __restrict__ partial, int nparts, int32_t margin, int32_t* __restrict__ bias,
    uint32_t* __restrict__ amax_bits, uint32_t* __restrict__ flags) {
    __shared__ uint32_t red[kAmaxThreads / 64];
    uint32_t m = strided_max<kAmaxThreads>(partial, nparts);
    m = block_max(m, red);
    if (threadIdx.x == 0) {
        const uint32_t a32 = canon_amax(DT == FP8_DT_BF16 ? (m << 16) : m);
        uint32_t fl;
        const int32_t b = bias_of<FMT>(a32, margin, &fl);
        *bias = b;
        if (amax_bits) *amax_bits = a32;
        if (flags) *flags = fl;
    }
}

template <int FMT>
__global__ void bias_from_amax_kernel(const uint32_t* __restrict__ amax_bits, int32_t margin,
                                      int32_t* __restrict__ bias, uint32_t* __restrict__ flags) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        uint32_t fl;
        *bias = bias_of<FMT>(*amax_bits, margin, &fl);
        if (flags) *flags = fl;
    }
}

// Workgroup tile: 128 rows x 128 columns, 256 threads.  Lane l of wave w owns
// rows r0 .. r0+7 (r0 = 8 (4 w + l / 16)) and columns c0 .. c0+7
// (c0 = 8 (l % 16)): each of its row loads is one 16-byte (bf16) or two
// 16-byte (fp32) accesses, 16 lanes covering 256 (512) contiguous bytes.
constexpr int kCastRows = 128, kCastCols = 128, kCastThreads = 256, kRpt = 8;


__device__ __forceinline__ uint32_t byte_of(uint32_t w, int j) { return (w >> (8 * j)) & 0xFFu; }

// One 128 x 128 tile (tile row tr, tile column tc) of the cast with bias b:
// codes to q (if given) and transposed codes to qT (if given).  With MAX, the
// largest magnitude pattern of the tile's elements (bf16: 15 bits, fp32: 31
// bits; 0 past the edges) is returned, valid in every thread after a block
// reduction by the caller.  Every thread of the block must call it (it
// synchronises through the LDS tile), and it leaves the LDS tile free for
// the next call.
// With ROWB, row r is cast with its own bias rowb[r] (clamped) instead of b.
// EDGE = false: every tile of the tensor is whole (rows and columns multiples
// of 128); the kernels that stream large tensors are built both ways, since
// the edge code costs registers and with them 1-2 % of the bandwidth, in the
// second pass of the quantise 10 % (4096 x 4096 fp32 without a prediction,
// 133 registers against 126: 32.4 us and 29.8).
// BULK = false: fp32 rows of whole tiles load as the compiler interleaves them
// with the conversions (see launch_cast_t).
template <int DT, int FMT, bool MAX, bool ROWB = false, bool EDGE = true, bool BULK = true>
__device__ __forceinline__ uint32_t cast_tile(const void* __restrict__ x, int64_t rows, int64_t cols,
                                              int64_t ldx, int b, uint8_t* __restrict__ q, int64_t ldq,
                                              uint8_t* __restrict__ qT, int64_t ldqT, int64_t tr,
                                              int64_t tc, uint8_t* __restrict__ tile,
                                              const int32_t* __restrict__ rowb = nullptr) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int chunk = lane & 15, g = lane >> 4;
    const int64_t R0 = tr * kCastRows, C0 = tc * kCastCols;
    const int lr = (w * 4 + g) * kRpt, lc = chunk * 8;
    const int64_t r0 = R0 + lr, c0 = C0 + lc;
    int bi[kRpt];  // bias of each of this lane's rows
#pragma unroll
    for (int i = 0; i < kRpt; ++i) bi[i] = ROWB ? clamp_bias(rowb[min(r0 + i, rows - 1)]) : b;

    uint32_t lo[kRpt], hi[kRpt];  // codes of columns c0..c0+3 and c0+4..c0+7, per row
    uint32_t mag = 0;
    // Rows past the last one read the last row again (not stored; a copy of
    // real elements cannot change the maximum), so only the columns of a
    // lane's block decide how it loads: eight whole columns, the last ones of
    // the row (one vector ending at the row's end, moved down, zeros beyond),
    // or those of a single row or of rows of fewer than eight columns (below);
    // lanes with no row at all load nothing.  One lane on a partial block used to go element by element, 64 guarded loads in a
    // row, and kept the whole launch waiting; transposed codes with an odd row
    // stride left as single bytes.  fp8_quantise of 301 x 4096: 13.0 -> 7.2 us;
    // 1531 x 4096 with transposed codes: 25.0 -> 12.9 us; whole tiles as before
    // (4096 x 11008 with both copies 36 us, 5.0 TB/s).
    const int64_t last = rows - 1;
    const int64_t left = EDGE ? cols - c0 : 8;  // columns of the row from c0 on
    const int nc = (int)min(cols, (int64_t)8);
    const bool whole = !EDGE || (R0 + kCastRows <= rows && C0 + kCastCols <= cols);  // of the tile: uniform
    int64_t at = (whole ? r0 : min(r0, last)) * ldx + c0;
    auto next_row = [&](int i) { at += whole || r0 + i < last ? ldx : 0; };
    // codes of eight elements of row i, and of four
    auto half_bf16 = [&](int i, uint32_t w0, uint32_t w1) {
        const uint32_t c = cast4_bf16<FMT>(w0, w1, bi[i]);
        if (__builtin_expect(!any_nan_bf16(w0, w1), 1)) return c;
        const uint32_t h[4] = {w0 & 0xFFFFu, w0 >> 16, w1 & 0xFFFFu, w1 >> 16};
        return nan_patch<FMT>(c, h);
    };
    auto half_f32 = [&](int i, const uint4& a) {
        const uint32_t c = cast4_f32<FMT>(a, bi[i]);
        if (__builtin_expect(((a.x | a.y | a.z | a.w) & 0x7F800000u) != 0x7F800000u, 1)) return c;
        const uint32_t h[4] = {f32_key(a.x), f32_key(a.y), f32_key(a.z), f32_key(a.w)};  // some exponent may be all ones
        return nan_patch<FMT>(c, h);
    };
    auto put_bf16 = [&](int i, const uint4& v) {
        lo[i] = cast4_bf16<FMT>(v.x, v.y, bi[i]);
        hi[i] = cast4_bf16<FMT>(v.z, v.w, bi[i]);
        if (__builtin_expect(any_nan_bf16(v.x, v.y) || any_nan_bf16(v.z, v.w), 0)) {
            const uint32_t h0[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
            const uint32_t h1[4] = {v.z & 0xFFFFu, v.z >> 16, v.w & 0xFFFFu, v.w >> 16};
            lo[i] = nan_patch<FMT>(lo[i], h0);
            hi[i] = nan_patch<FMT>(hi[i], h1);
        }
    };
    auto put_f32 = [&](int i, const uint4& a, const uint4& bb) {
        if (MAX) mag = fold_f32(fold_f32(mag, a), bb);
        lo[i] = cast4_f32<FMT>(a, bi[i]);
        hi[i] = cast4_f32<FMT>(bb, bi[i]);
        const uint32_t m = (a.x | a.y | a.z | a.w | bb.x | bb.y | bb.z | bb.w) & 0x7F800000u;
        if (__builtin_expect(m == 0x7F800000u, 0)) {  // some exponent field may be all ones
            const uint32_t h0[4] = {f32_key(a.x), f32_key(a.y), f32_key(a.z), f32_key(a.w)};
            const uint32_t h1[4] = {f32_key(bb.x), f32_key(bb.y), f32_key(bb.z), f32_key(bb.w)};
            lo[i] = nan_patch<FMT>(lo[i], h0);
            hi[i] = nan_patch<FMT>(hi[i], h1);
        }
    };
    if (EDGE && rows > 1 && r0 >= rows) {
#pragma unroll
        for (int i = 0; i < kRpt; ++i) lo[i] = hi[i] = 0;
    } else if (!EDGE || (cols >= 8 && rows > 1)) {
        const int drop = whole || left >= 8 ? 0 : left > 0 ? (int)(8 - left) : 8;  // elements moved out
        at -= drop;
        if (DT == FP8_DT_BF16) {
            uint4 v[kRpt];
            if (whole) {
#pragma unroll
                for (int i = 0; i < kRpt; ++i) v[i] = ld_stream((const uint16_t*)x + at + i * ldx);
            } else {
#pragma unroll
                for (int i = 0; i < kRpt; ++i) {
                    v[i] = ld_stream((const uint16_t*)x + (left > 0 ? at : 0));
                    next_row(i);
                }
            }
            if (drop) {
#pragma unroll
                for (int i = 0; i < kRpt; ++i) v[i] = shr128(v[i], 16 * drop);
            }
            if (MAX) {
                us2 mm = {0, 0};
#pragma unroll
                for (int i = 0; i < kRpt; ++i) mm = fold_bf16(mm, v[i]);
                mag = max((uint32_t)mm.x, (uint32_t)mm.y);
            }
#pragma unroll
            for (int i = 0; i < kRpt; ++i) put_bf16(i, v[i]);
        } else if ((MAX || !BULK) && !EDGE) {
            // the compiler interleaves loads and conversions (see below)
#pragma unroll
            for (int i = 0; i < kRpt; ++i) {
                const uint32_t* p = (const uint32_t*)x + (r0 + i) * ldx + c0;
                const uint4 a = ld_stream(p), bb = ld_stream(p + 4);
                put_f32(i, a, bb);
            }
        } else {
            // All rows' loads in flight at once pay in the plain cast and in
            // small tensors, but cost the quantise of whole tiles, which also
            // folds the maximum, its occupancy (5.05 -> 4.91 TB/s).
            uint4 va[kRpt], vb[kRpt];
            const int64_t at0 = at;
            auto load = [&](int i) {
                const uint32_t* p = (const uint32_t*)x + (whole ? at0 + i * ldx : left > 0 ? at : 0);
                va[i] = ld_stream(p);
                vb[i] = ld_stream(p + 4);
                if (!whole) next_row(i);
            };
            if (!MAX || (EDGE && !whole)) {
#pragma unroll
                for (int i = 0; i < kRpt; ++i) load(i);
            }
#pragma unroll
            for (int i = 0; i < kRpt; ++i) {
                if (MAX && whole) load(i);
                uint4 a = va[i], bb = vb[i];
                if (drop) {
                    if (drop & 8) a = bb = make_uint4(0u, 0u, 0u, 0u);
                    if (drop & 4) a = bb, bb = make_uint4(0u, 0u, 0u, 0u);
                    if (drop & 2) a = make_uint4(a.z, a.w, bb.x, bb.y), bb = make_uint4(bb.z, bb.w, 0u, 0u);
                    if (drop & 1) a = make_uint4(a.y, a.z, a.w, bb.x), bb = make_uint4(bb.y, bb.z, bb.w, 0u);
                }
                put_f32(i, a, bb);
            }
        }
    } else if (rows == 1) {
        // A single row (a vector, a token): its 16 lanes read it once, where
        // every lane of a partial tile reads eight rows (cast of 1 x 80000 fp32:
        // 8.9 -> 2.8 us, 1 x 4096 bf16: 4.0 -> 2.5).  Columns past the last one read it again and become
        // zero, so that the loads need no branch of a lane.
#pragma unroll
        for (int i = 0; i < kRpt; ++i) lo[i] = hi[i] = 0;
        if (lr == 0 && left > 0) {
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t c = min(c0 + j, cols - 1);
                e[j] = DT == FP8_DT_BF16 ? ((const uint16_t*)x)[c] : ((const uint32_t*)x)[c];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = j < left ? e[j] : 0u;
            if (DT == FP8_DT_BF16) {
                const uint4 v = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
                if (MAX) {
                    const us2 mm = fold_bf16(us2{0, 0}, v);
                    mag = max((uint32_t)mm.x, (uint32_t)mm.y);
                }
                put_bf16(0, v);
            } else {
                put_f32(0, make_uint4(e[0], e[1], e[2], e[3]), make_uint4(e[4], e[5], e[6], e[7]));
            }
        }
    } else if (nc > 4) {
        // Rows of five to seven columns: eight elements from the row's start on
        // (in the last rows the tensor's last eight, moved down), those past
        // the row's end zero.
#pragma unroll
        for (int i = 0; i < kRpt; ++i) lo[i] = hi[i] = 0;
        if (left > 0) {
            const int64_t end8 = last * ldx + cols - 8;  // two rows or more: at least 2 cols - 8 > 0
            us2 mm = {0, 0};
#pragma unroll
            for (int i0 = 0; i0 < kRpt; i0 += 4) {  // four rows in flight: no more registers than the other branches
                uint4 va[4], vb[4];
                int moved[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t from = min(at, end8);
                    moved[k] = (int)(at - from);
                    if (DT == FP8_DT_BF16) {
                        va[k] = ld_stream((const uint16_t*)x + from);
                    } else {
                        va[k] = ld_stream((const uint32_t*)x + from);
                        vb[k] = ld_stream((const uint32_t*)x + from + 4);
                    }
                    next_row(i0 + k);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (DT == FP8_DT_BF16) {
                        auto keep = [&](int w) { return nc > 2 * w + 1 ? ~0u : nc > 2 * w ? 0xFFFFu : 0u; };
                        uint4 v = moved[k] ? shr128(va[k], 16 * moved[k]) : va[k];
                        v = make_uint4(v.x & keep(0), v.y & keep(1), v.z & keep(2), v.w & keep(3));
                        if (MAX) mm = fold_bf16(mm, v);
                        put_bf16(i0 + k, v);
                    } else {
                        uint4 a = va[k], bb = vb[k];
                        if (moved[k] & 4) a = bb;  // what is left of bb lies past the row's end
                        if (moved[k] & 2) a = make_uint4(a.z, a.w, bb.x, bb.y), bb = make_uint4(bb.z, bb.w, 0u, 0u);
                        if (moved[k] & 1) a = make_uint4(a.y, a.z, a.w, bb.x), bb = make_uint4(bb.y, bb.z, bb.w, 0u);
                        a = make_uint4(a.x, nc > 1 ? a.y : 0u, nc > 2 ? a.z : 0u, nc > 3 ? a.w : 0u);
                        bb = make_uint4(nc > 4 ? bb.x : 0u, nc > 5 ? bb.y : 0u, nc > 6 ? bb.z : 0u, 0u);
                        put_f32(i0 + k, a, bb);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MAX && DT == FP8_DT_BF16) mag = max((uint32_t)mm.x, (uint32_t)mm.y);
        }
    } else {
        // Rows of one to four columns: their elements, all loads in flight (cast
        // of 10^6 x 4 bf16 one element after another 52 us, fp32 54; now 25 and
        // 32; with the vectors of the branch above 38 and 48).
#pragma unroll
        for (int i = 0; i < kRpt; ++i) lo[i] = hi[i] = 0;
        if (left > 0) {
            uint32_t e[kRpt][4];
            int64_t row[kRpt];
#pragma unroll
            for (int i = 0; i < kRpt; ++i) {
                row[i] = at;
                next_row(i);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int i = 0; i < kRpt; ++i) e[i][j] = 0;
                if (j < nc) {
#pragma unroll
                    for (int i = 0; i < kRpt; ++i)
                        e[i][j] = DT == FP8_DT_BF16 ? ((const uint16_t*)x)[row[i] + j] : ((const uint32_t*)x)[row[i] + j];
                }
            }
#pragma unroll
            for (int i = 0; i < kRpt; ++i) {
                if (DT == FP8_DT_BF16) {
                    const uint32_t w0 = e[i][0] | (e[i][1] << 16), w1 = e[i][2] | (e[i][3] << 16);
                    if (MAX) {
                        const us2 mm = fold_bf16(us2{0, 0}, make_uint4(w0, w1, 0u, 0u));
                        mag = max(mag, max((uint32_t)mm.x, (uint32_t)mm.y));
                    }
                    lo[i] = half_bf16(i, w0, w1);
                } else {
                    const uint4 a = make_uint4(e[i][0], e[i][1], e[i][2], e[i][3]);
                    if (MAX) mag = fold_f32(mag, a);
                    lo[i] = half_f32(i, a);
                }
            }
        }
    }

    if (q) {
        uint8_t* o = q + r0 * ldq + c0;
        if (whole) {
#pragma unroll
            for (int i = 0; i < kRpt; ++i) st8_any(o + i * ldq, lo[i], hi[i]);
        } else {
#pragma unroll
            for (int i = 0; i < kRpt; ++i, o += ldq) {
                if (r0 + i >= rows) break;
                if (left >= 8) {
                    st8_any(o, lo[i], hi[i]);
                } else {
                    for (int j = 0; j < 8; ++j)
                        if (j < left) o[j] = (uint8_t)byte_of(j < 4 ? lo[i] : hi[i], j & 3);
                }
            }
        }
    }

    if (qT) {
        // Column c0 + j of this lane's 8x8 block, rows r0..r0+7, as 8 bytes at
        // row offset lr of transposed row lc + j; 16-byte chunks of a
        // transposed row are XOR-swizzled with the column block.
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t* src = j < 4 ? lo : hi;
            const int jj = j & 3;
            const uint32_t w0 = byte_of(src[0], jj) | (byte_of(src[1], jj) << 8) | (byte_of(src[2], jj) << 16) |
                                (byte_of(src[3], jj) << 24);
            const uint32_t w1 = byte_of(src[4], jj) | (byte_of(src[5], jj) << 8) | (byte_of(src[6], jj) << 16) |
                                (byte_of(src[7], jj) << 24);
            const int cl = lc + j;
            const int off = cl * kCastRows + ((((lr >> 4) ^ (cl >> 3)) & 7) << 4) + (lr & 15);
            *(uint2*)(tile + off) = make_uint2(w0, w1);
        }
        __syncthreads();
        // 128 transposed rows x 8 chunks of 16 bytes = 1024 chunks, four per thread.
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int idx = threadIdx.x + h * kCastThreads;
            const int cl = idx >> 3, qq = idx & 7;
            const int64_t c = C0 + cl;
            const int64_t rr = R0 + qq * 16;
            if (EDGE && (c >= cols || rr >= rows)) continue;
            const uint4 v = *(const uint4*)(tile + cl * kCastRows + (((qq ^ (cl >> 3)) & 7) << 4));
            uint8_t* dst = qT + c * ldqT + rr;
            if (!EDGE || rr + 16 <= rows) {
                st16_any(dst, v);
            } else {
                const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                for (int t = 0; t < 16 && rr + t < rows; ++t) dst[t] = (uint8_t)byte_of(wv[t >> 2], t & 3);
            }
        }
        __syncthreads();  // the tile may be rewritten by the next call
    }
    return mag;
}


template <int DT, int FMT, bool EDGE, bool BULK>
__global__ __launch_bounds__(kCastThreads) void cast_kernel(
    const void* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx,
    const int32_t* __restrict__ bias_p, uint8_t* __restrict__ q, int64_t ldq,
    uint8_t* __restrict__ qT, int64_t ldqT, int64_t tiles_c) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    const int b = clamp_bias(*bias_p);
    cast_tile<DT, FMT, false, false, EDGE, BULK>(x, rows, cols, ldx, b, q, ldq, qT, ldqT, blockIdx.x / tiles_c,
                                                 blockIdx.x % tiles_c, tile);
}

// ------------------------------------------------- quantise: amax + bias + cast
// Pass 1 (quant_pass1_kernel), one workgroup per tile: the largest magnitude
// pattern of the tile goes to parts[tile]; with CAST the tile is also cast with
// the predicted bias (clamped), which block 0 records in *used.
// Pass 2 (quant_pass2_kernel): every workgroup reduces parts[] and evaluates
// Eq. 3; block 0 writes bias, amax and flags.  If pass 1 did not cast, or cast
// with a bias other than the exact one, the workgroups recast all ncast tiles
// (grid-stride) with the exact bias; otherwise the codes of pass 1 are already
// those of the exact bias and nothing more is written.  parts[] may come from
// another producer of the same tensor (a matmul epilogue) with its own tiling.
template <int DT, int FMT, bool CAST, bool EDGE>
__global__ __launch_bounds__(kCastThreads) void quant_pass1_kernel(
    const void* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx,
    const int32_t* __restrict__ bias_pred, int32_t* __restrict__ used, uint32_t* __restrict__ parts,
    uint8_t* __restrict__ q, int64_t ldq, uint8_t* __restrict__ qT, int64_t ldqT, int64_t tiles_c) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    __shared__ uint32_t red[kCastThreads / 64];
    int b = 0;
    if (CAST) {
        b = clamp_bias(*bias_pred);
        if (blockIdx.x == 0 && threadIdx.x == 0) *used = b;
    }
    const uint32_t m = cast_tile<DT, FMT, true, false, EDGE>(x, rows, cols, ldx, b, CAST ? q : nullptr, ldq,
                                                CAST ? qT : nullptr, ldqT, blockIdx.x / tiles_c,
                                                blockIdx.x % tiles_c, tile);
    const uint32_t bm = block_max(m, red);
    if (threadIdx.x == 0) parts[blockIdx.x] = bm;
}

// Both passes in one launch for a small tensor: every workgroup takes the
// maximum of the whole tensor (from L2 after the first read), so it has the
// exact bias without waiting for the others, and casts one tile; block 0 writes bias, amax and flags, and into *used what the prediction was
// (nothing is cast with it).  The tensor is read as rows of vpr vectors (the
// last one of a row ends at its end; overlaps do not change a maximum); magic
// divides a vector index by vpr.
template <int DT, int FMT>
__global__ __launch_bounds__(kCastThreads) void quant_small_kernel(
    const void* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx, int cols1, int vpr, int nvec, uint32_t magic,
    int32_t margin, const int32_t* bias_pred, int32_t* __restrict__ used, int32_t* bias,
    uint32_t* __restrict__ amax_bits, uint32_t* __restrict__ flags, uint8_t* __restrict__ q, int64_t ldq,
    uint8_t* __restrict__ qT, int64_t ldqT, int tiles_c) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    __shared__ uint32_t red[kCastThreads / 64];
    constexpr int per = DT == FP8_DT_BF16 ? 8 : 4, kL = 8;
    uint32_t m = 0;
    us2 mm = {0, 0};
    for (int i = threadIdx.x; i < nvec; i += kL * kCastThreads) {
        uint4 v[kL];
#pragma unroll
        for (int l = 0; l < kL; ++l) {
            const int iv = min(i + l * kCastThreads, nvec - 1);
            const int r = (int)__umulhi((uint32_t)iv, magic), c = min((iv - r * vpr) * per, cols1 - per);
            v[l] = ld16_any((const char*)x + (r * ldx + c) * (DT == FP8_DT_BF16 ? 2 : 4));
        }
        __builtin_amdgcn_sched_barrier(0);  // all loads issue before the first use
#pragma unroll
        for (int l = 0; l < kL; ++l) {
            if (DT == FP8_DT_BF16) mm = fold_bf16(mm, v[l]);
            else m = fold_f32(m, v[l]);
        }
    }
    if (DT == FP8_DT_BF16) m = max((uint32_t)mm.x, (uint32_t)mm.y);
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kCastThreads / 64; ++w) m = max(m, red[w]);
    const uint32_t a32 = canon_amax(DT == FP8_DT_BF16 ? (m << 16) : m);
    uint32_t fl;
    const int32_t bx = bias_of<FMT>(a32, margin, &fl);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (bias_pred) *used = clamp_bias(*bias_pred);  // may be the same word as *bias
        *bias = bx;
        if (amax_bits) *amax_bits = a32;
        if (flags) *flags = fl;
    }
    cast_tile<DT, FMT, false>(x, rows, cols, ldx, clamp_bias(bx), q, ldq, qT, ldqT, blockIdx.x / tiles_c,
                              blockIdx.x % tiles_c, tile);
}

// Pass 2 of one tensor as workgroup bid of nb: see quant_pass2_kernel.
template <int DT, int FMT, bool EDGE>
__device__ __forceinline__ void quant_pass2_body(
    int bid, int nb, uint8_t* tile, uint32_t* red, uint32_t& amax_s, const void* __restrict__ x,
    int64_t rows, int64_t cols, int64_t ldx, const uint32_t* __restrict__ parts, int nparts,
    const int32_t* __restrict__ used, int have_used, int32_t margin, int32_t* __restrict__ bias,
    uint32_t* __restrict__ amax_bits, uint32_t* __restrict__ flags, uint8_t* __restrict__ q, int64_t ldq,
    uint8_t* __restrict__ qT, int64_t ldqT, int64_t tiles_c, int64_t ncast) {
    uint32_t m = strided_max<kCastThreads>(parts, nparts);
    m = block_max(m, red);
    if (threadIdx.x == 0) amax_s = m;
    __syncthreads();
    const uint32_t a32 = canon_amax(DT == FP8_DT_BF16 ? (amax_s << 16) : amax_s);
    uint32_t fl;
    const int32_t bx = bias_of<FMT>(a32, margin, &fl);
    if (bid == 0 && threadIdx.x == 0) {
        *bias = bx;
        if (amax_bits) *amax_bits = a32;
        if (flags) *flags = fl;
    }
    const int b = clamp_bias(bx);
    if (have_used && *used == b) return;  // pass 1 already wrote these codes
    for (int64_t t = bid; t < ncast; t += nb)
        cast_tile<DT, FMT, false, false, EDGE>(x, rows, cols, ldx, b, q, ldq, qT, ldqT, t / tiles_c, t % tiles_c, tile);
}

template <int DT, int FMT, bool EDGE>
__global__ __launch_bounds__(kCastThreads) void quant_pass2_kernel(
    const void* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx,
    const uint32_t* __restrict__ parts, int nparts, const int32_t* __restrict__ used, int have_used,
    int32_t margin, int32_t* __restrict__ bias, uint32_t* __restrict__ amax_bits,
    uint32_t* __restrict__ flags, uint8_t* __restrict__ q, int64_t ldq, uint8_t* __restrict__ qT,
    int64_t ldqT, int64_t tiles_c, int64_t ncast) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    __shared__ uint32_t red[kCastThreads / 64];
    __shared__ uint32_t amax_s;
    quant_pass2_body<DT, FMT, EDGE>(blockIdx.x, gridDim.x, tile, red, amax_s, x, rows, cols, ldx, parts, nparts, used,
                                    have_used, margin, bias, amax_bits, flags, q, ldq, qT, ldqT, tiles_c, ncast);
}

// ------------------------------------------------ delayed scaling
// The second launch of fp8_quantise_delayed (one workgroup): the tensor's amax
// from the tile maxima of pass 1 (cast with the bias in *bias, recorded in
// *used), whether those codes clipped (amax * 2^used > max_num, i.e. used is
// above the tensor's own Eq. 3 bias), the amax appended to the history ring
// at *count % hlen, and the bias of the next call: Eq. 3 of the largest amax
// in the history, minus the margin.  History words are amax bit patterns with
// the sign clear (canonical NaN 0x7FC00000 largest), so their integer maximum
// is the largest amax.  Slot *count % hlen is left out of the history
// reduction and replaced by this tensor's amax, so no thread reads the word
// thread 0 writes.
template <int DT, int FMT>
__global__ __launch_bounds__(kCastThreads) void quant_delayed_finish_kernel(
    const uint32_t* __restrict__ parts, int nparts, const int32_t* __restrict__ used, int32_t margin,
    uint32_t* __restrict__ history, int hlen, uint32_t* __restrict__ count, int32_t* __restrict__ bias,
    uint32_t* __restrict__ amax_bits, uint32_t* __restrict__ flags) {
    __shared__ uint32_t red[kCastThreads / 64];
    __shared__ uint32_t slot_s;
    uint32_t m = strided_max<kCastThreads>(parts, nparts);
    m = block_max(m, red);
    if (threadIdx.x == 0) slot_s = *count;
    __syncthreads();
    const uint32_t c = slot_s;
    const int slot = (int)(c % (uint32_t)hlen);
    uint32_t h = 0;
    for (int i = threadIdx.x; i < hlen; i += kCastThreads)
        if (i != slot) h = max(h, history[i]);
    __syncthreads();  // red[] is reused
    h = block_max(h, red);
    if (threadIdx.x == 0) {
        const uint32_t a32 = canon_amax(DT == FP8_DT_BF16 ? (m << 16) : m);
        uint32_t fl;
        const int32_t own = bias_of<FMT>(a32, 0, &fl);
        if (fl == 0u && nparts > 0 && *used > own) fl = FP8_FLAG_SATURATED;
        history[slot] = a32;
        *count = c + 1u;
        uint32_t fl_next;
        *bias = bias_of<FMT>(max(h, a32), margin, &fl_next);
        if (amax_bits) *amax_bits = a32;
        if (flags) *flags = fl;
    }
}

// ------------------------------------------------ quantise several tensors
// fp8_quantise of up to kQBatch tensors of one element type and format in one
// pass-1 launch and one pass-2 launch: workgroups [t0[i], t0[i+1]) of pass 1
// are tensor i's tiles, workgroups [p0[i], p0[i+1]) of pass 2 its finishing
// workgroups; each tensor keeps its own workspace (used word + tile maxima),
// so the bits are those of separate calls.
struct QBatch {
    int n;
    int64_t t0[kQBatch + 1], p0[kQBatch + 1];
    const void* x[kQBatch];
    int64_t rows[kQBatch], cols[kQBatch], ldx[kQBatch], tiles_c[kQBatch];
    const int32_t* pred[kQBatch];
    int32_t* bias[kQBatch];
    uint32_t* amax[kQBatch];
    uint32_t* flags[kQBatch];
    uint8_t* q[kQBatch];
    int64_t ldq[kQBatch];
    uint8_t* qT[kQBatch];
    int64_t ldqT[kQBatch];
    uint32_t* ws[kQBatch];
};

__device__ __forceinline__ int batch_slot(const int64_t* start, int n, int64_t b) {
    int i = 0;
    while (i + 1 < n && b >= start[i + 1]) ++i;
    return i;
}

template <int DT, int FMT, bool CAST, bool EDGE>
__global__ __launch_bounds__(kCastThreads) void quant_pass1_batch_kernel(QBatch qb) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    __shared__ uint32_t red[kCastThreads / 64];
    const int i = batch_slot(qb.t0, qb.n, blockIdx.x);
    const int64_t t = (int64_t)blockIdx.x - qb.t0[i];
    int b = 0;
    if (CAST) {
        b = clamp_bias(*qb.pred[i]);
        if (t == 0 && threadIdx.x == 0) *(int32_t*)qb.ws[i] = b;
    }
    const uint32_t m = cast_tile<DT, FMT, true, false, EDGE>(qb.x[i], qb.rows[i], qb.cols[i], qb.ldx[i], b, CAST ? qb.q[i] : nullptr,
                                                qb.ldq[i], CAST ? qb.qT[i] : nullptr, qb.ldqT[i], t / qb.tiles_c[i],
                                                t % qb.tiles_c[i], tile);
    const uint32_t bm = block_max(m, red);
    if (threadIdx.x == 0) qb.ws[i][1 + t] = bm;
}

template <int DT, int FMT, bool EDGE>
__global__ __launch_bounds__(kCastThreads) void quant_pass2_batch_kernel(QBatch qb, int32_t margin, int have_used) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    __shared__ uint32_t red[kCastThreads / 64];
    __shared__ uint32_t amax_s;
    const int i = batch_slot(qb.p0, qb.n, blockIdx.x);
    const int64_t ntiles = qb.t0[i + 1] - qb.t0[i];
    quant_pass2_body<DT, FMT, EDGE>((int)(blockIdx.x - qb.p0[i]), (int)(qb.p0[i + 1] - qb.p0[i]), tile, red, amax_s,
                                    qb.x[i], qb.rows[i], qb.cols[i], qb.ldx[i], qb.ws[i] + 1, (int)ntiles,
                                    (const int32_t*)qb.ws[i], have_used, margin, qb.bias[i], qb.amax[i], qb.flags[i],
                                    qb.q[i], qb.ldq[i], qb.qT[i], qb.ldqT[i], qb.tiles_c[i], ntiles);
}

// fn(true_type) when some tile of a rows x cols tensor is partial.
bool has_edge(int64_t rows, int64_t cols) { return rows % kCastRows != 0 || cols % kCastCols != 0; }
template <typename Fn>
void with_edge(bool edge, Fn&& fn) {
    if (edge) fn(std::true_type{}); else fn(std::false_type{});
}

// LDS that a launch asks for beyond its tile, to hold five workgroups of a
// compute unit instead of seven, where bf16 rows end inside a tile: their codes
// leave as partial lines, which more tiles in flight evict before they are whole
// (cast of 8192 x 4095 43.9 -> 38.7 us, quantise 46.9 -> 41.2; rows of whole
// tiles and narrower tensors lose by it or do not care).
template <int DT>
constexpr unsigned spare_lds(int64_t cols) {
    return DT == FP8_DT_BF16 && cols > kCastCols && cols % kCastCols != 0 ? 16u << 10 : 0u;
}

// fp32 casts of whole tiles with all of a lane's loads in flight at once (90
// registers), or interleaved with the conversions (about 60).  All at once
// where few tiles leave the latency open (2048 x 4096: 9.3 us against 10.1) and
// where the tensor comes from HBM and rows of codes leave (4096 x 11008 47.8
// against 50.2, with both copies 58.1 against 60.9); interleaved from about two
// tiles per compute unit to what the last-level cache holds (4096 x 8192 35.0
// against 31.9, both copies 42.7 against 37.8; 2048 x 5120 12.4 against 11.8)
// and for transposed codes alone (8192 x 8192 72.5 against 70.1).
constexpr int64_t kBulkTiles = 512, kBulkTilesHbm = 2048;

template <int DT, int FMT>
void launch_cast_t(const void* x, int64_t rows, int64_t cols, int64_t ldx, const int32_t* bias,
                   uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT, hipStream_t s) {
    const int64_t tiles_r = (rows + kCastRows - 1) / kCastRows;
    const int64_t tiles_c = (cols + kCastCols - 1) / kCastCols, ntiles = tiles_r * tiles_c;
    const bool edge = has_edge(rows, cols);
    if (DT == FP8_DT_F32 && !edge && ntiles > kBulkTiles && (ntiles <= kBulkTilesHbm || !q)) {
        hipLaunchKernelGGL((cast_kernel<DT, FMT, false, DT != FP8_DT_F32>), dim3((unsigned)ntiles), dim3(kCastThreads), 0, s,
                           x, rows, cols, ldx, bias, q, ldq, qT, ldqT, tiles_c);
        return;
    }
    with_edge(edge, [&](auto E) {
        hipLaunchKernelGGL((cast_kernel<DT, FMT, decltype(E)::value, true>), dim3((unsigned)ntiles), dim3(kCastThreads),
                           spare_lds<DT>(cols), s,
                           x, rows, cols, ldx, bias, q, ldq, qT, ldqT, tiles_c);
    });
}

constexpr int kQuantPass2MaxBlocks = 1024;

// Largest tensor (bytes) quantised in one launch: 1 x 4096 bf16 takes 3.3 us
// against 5.8 with two launches, 16 x 4096 (128 KiB) 5.6 against 7.1, 16 x 8192
// (256 KiB) 8.3 against 7.1 (a workgroup pulls about 60 GB/s from L2).
constexpr int64_t kSmallBytes = 160 << 10;

template <int DT, int FMT>
void launch_quantise_t(const void* x, int64_t rows, int64_t cols, int64_t ldx, int32_t margin,
                       const int32_t* bias_pred, int32_t* bias, uint32_t* amax_bits, uint32_t* flags,
                       uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT, uint32_t* ws,
                       hipStream_t s) {
    const int64_t tiles_r = (rows + kCastRows - 1) / kCastRows;
    const int64_t tiles_c = (cols + kCastCols - 1) / kCastCols;
    const int64_t ntiles = tiles_r * tiles_c;
    int32_t* used = (int32_t*)ws;
    uint32_t* parts = ws + 1;
    constexpr int per = DT == FP8_DT_BF16 ? 8 : 4;
    if (cols >= 8 && (ldx == cols || cols > per) && rows * cols * (16 / per) <= kSmallBytes) {
        // dense: one row of all elements
        const int rows1 = ldx == cols ? 1 : (int)rows, cols1 = (int)(ldx == cols ? rows * cols : cols);
        const int vpr = (cols1 + per - 1) / per;
        const uint32_t magic = rows1 == 1 ? 0u : 0xFFFFFFFFu / (uint32_t)vpr + 1u;
        hipLaunchKernelGGL((quant_small_kernel<DT, FMT>), dim3((unsigned)ntiles), dim3(kCastThreads), 0, s, x, rows, cols,
                           ldx, cols1, vpr, rows1 * vpr, magic, margin, bias_pred, used, bias, amax_bits, flags, q, ldq,
                           qT, ldqT, (int)tiles_c);
        return;
    }
    with_edge(has_edge(rows, cols), [&](auto E) {
        constexpr bool kE = decltype(E)::value;
        if (bias_pred)
            hipLaunchKernelGGL((quant_pass1_kernel<DT, FMT, true, kE>), dim3((unsigned)ntiles), dim3(kCastThreads),
                               spare_lds<DT>(cols), s,
                               x, rows, cols, ldx, bias_pred, used, parts, q, ldq, qT, ldqT, tiles_c);
        else
            hipLaunchKernelGGL((quant_pass1_kernel<DT, FMT, false, kE>), dim3((unsigned)ntiles), dim3(kCastThreads), 0, s,
                               x, rows, cols, ldx, bias_pred, used, parts, q, ldq, qT, ldqT, tiles_c);
        const int nb2 = (int)(ntiles < kQuantPass2MaxBlocks ? ntiles : kQuantPass2MaxBlocks);
        hipLaunchKernelGGL((quant_pass2_kernel<DT, FMT, kE>), dim3(nb2), dim3(kCastThreads), 0, s, x, rows, cols, ldx,
                           parts, (int)ntiles, used, bias_pred ? 1 : 0, margin, bias, amax_bits, flags, q, ldq,
                           qT, ldqT, tiles_c, ntiles);
    });
}

template <int DT, int FMT>
void launch_quantise_batch_t(int n, const QuantDesc* d, int32_t margin, hipStream_t s) {
    QBatch qb{};
    qb.n = n;
    bool pred = false, edge = false;
    for (int i = 0; i < n; ++i) {
        edge = edge || has_edge(d[i].rows, d[i].cols);
        const int64_t tiles_c = (d[i].cols + kCastCols - 1) / kCastCols;
        const int64_t ntiles = ((d[i].rows + kCastRows - 1) / kCastRows) * tiles_c;
        qb.t0[i + 1] = qb.t0[i] + ntiles;
        qb.p0[i + 1] = qb.p0[i] + (ntiles < kQuantPass2MaxBlocks ? ntiles : kQuantPass2MaxBlocks);
        qb.x[i] = d[i].x;
        qb.rows[i] = d[i].rows;
        qb.cols[i] = d[i].cols;
        qb.ldx[i] = d[i].ldx;
        qb.tiles_c[i] = tiles_c;
        qb.pred[i] = d[i].pred;
        qb.bias[i] = d[i].bias;
        qb.amax[i] = d[i].amax;
        qb.flags[i] = d[i].flags;
        qb.q[i] = d[i].q;
        qb.ldq[i] = d[i].ldq;
        qb.qT[i] = d[i].qT;
        qb.ldqT[i] = d[i].ldqT;
        qb.ws[i] = d[i].ws;
        pred = d[i].pred != nullptr;
    }
    with_edge(edge, [&](auto E) {
        constexpr bool kE = decltype(E)::value;
        if (pred)
            hipLaunchKernelGGL((quant_pass1_batch_kernel<DT, FMT, true, kE>), dim3((unsigned)qb.t0[n]), dim3(kCastThreads), 0,
                               s, qb);
        else
            hipLaunchKernelGGL((quant_pass1_batch_kernel<DT, FMT, false, kE>), dim3((unsigned)qb.t0[n]),
                               dim3(kCastThreads), 0, s, qb);
        hipLaunchKernelGGL((quant_pass2_batch_kernel<DT, FMT, kE>), dim3((unsigned)qb.p0[n]), dim3(kCastThreads), 0, s, qb,
                           margin, pred ? 1 : 0);
    });
}

template <int DT, int FMT>
void launch_quant_check_t(const void* x, int64_t rows, int64_t cols, int64_t ldx, int32_t margin,
                          const uint32_t* parts, int nparts, const int32_t* used, int32_t* bias,
                          uint32_t* amax_bits, uint32_t* flags, uint8_t* q, int64_t ldq, uint8_t* qT,
                          int64_t ldqT, hipStream_t s) {
    const int64_t tiles_c = (cols + kCastCols - 1) / kCastCols;
    const int64_t ncast = ((rows + kCastRows - 1) / kCastRows) * tiles_c;
    const int nb2 = (int)(ncast < kQuantPass2MaxBlocks ? ncast : kQuantPass2MaxBlocks);
    with_edge(has_edge(rows, cols), [&](auto E) {
        hipLaunchKernelGGL((quant_pass2_kernel<DT, FMT, decltype(E)::value>), dim3(nb2), dim3(kCastThreads), 0, s, x, rows,
                           cols, ldx, parts, nparts, used, 1, margin, bias, amax_bits, flags, q, ldq, qT, ldqT, tiles_c,
                           ncast);
    });
}

template <int DT, int FMT>
void launch_quantise_delayed_t(const void* x, int64_t rows, int64_t cols, int64_t ldx, int32_t margin, int32_t* bias,
                               uint32_t* history, int hlen, uint32_t* count, uint32_t* amax_bits, uint32_t* flags,
                               uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT, uint32_t* ws, hipStream_t s) {
    const int64_t tiles_r = (rows + kCastRows - 1) / kCastRows;
    const int64_t tiles_c = (cols + kCastCols - 1) / kCastCols;
    const int64_t ntiles = tiles_r * tiles_c;
    int32_t* used = (int32_t*)ws;
    uint32_t* parts = ws + 1;
    if (ntiles > 0) {
        with_edge(has_edge(rows, cols), [&](auto E) {
            hipLaunchKernelGGL((quant_pass1_kernel<DT, FMT, true, decltype(E)::value>), dim3((unsigned)ntiles),
                               dim3(kCastThreads), spare_lds<DT>(cols), s, x, rows, cols, ldx, bias, used, parts, q, ldq, qT, ldqT, tiles_c);
        });
    }
    hipLaunchKernelGGL((quant_delayed_finish_kernel<DT, FMT>), dim3(1), dim3(kCastThreads), 0, s, parts, (int)ntiles,
                       used, margin, history, hlen, count, bias, amax_bits, flags);
}

// Host dispatch of (element type, format) to kernel template arguments.
template <int V> using IC = std::integral_constant<int, V>;

template <typename Fn>
void with_fmt(int fmt, Fn&& fn) {
    switch (fmt) {
        case FP8_E4M3: fn(IC<FP8_E4M3>{}); break;
        case FP8_E5M2: fn(IC<FP8_E5M2>{}); break;
        case FP8_E4_A: fn(IC<FP8_E4_A>{}); break;
        default: fn(IC<FP8_E5_A>{}); break;
    }
}

template <typename Fn>
void with_dt_fmt(int dt, int fmt, Fn&& fn) {
    if (dt == FP8_DT_BF16)
        with_fmt(fmt, [&](auto F) { fn(IC<FP8_DT_BF16>{}, F); });
    else
        with_fmt(fmt, [&](auto F) { fn(IC<FP8_DT_F32>{}, F); });
}


// ------------------------------------------- segments: one bias per row group
__global__ void fill_words_kernel(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Segment s holds rows offsets[s] <= r < offsets[s + 1] (one data sample or
// micro-batch).  Three launches: the largest magnitude pattern of every row,
// written where its bias will be; per segment (one workgroup) the maximum of
// its rows, Eq. 3, and the bias over the rows' words; the cast.  Offsets are
// clamped to the rows, so whatever they hold no access leaves the buffers.
// Before, the row maxima went to per-segment words through atomics: a launch
// to clear the words first, and rows read one vector at a time.  2151 x 4096
// in three segments: 23.3 -> 15.3 us; 100000 x 64: 300 -> 45 us.
constexpr int kRowWaves = 4;  // rows per workgroup of the first launch, one wave each

template <int DT>
__global__ __launch_bounds__(64 * kRowWaves) void row_max_kernel(const void* __restrict__ x, int64_t rows, int64_t cols,
                                                                 int64_t ldx, uint32_t* __restrict__ rmax) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * kRowWaves + (threadIdx.x >> 6);
    if (r >= rows) return;
    constexpr int per = DT == FP8_DT_BF16 ? 8 : 4, esz = 16 / per, kL = 8;
    const char* p = (const char*)x + r * ldx * esz;
    uint32_t m = 0;
    us2 mm = {0, 0};
    if (cols >= per) {  // vectors past the row end re-read its last one
        for (int64_t c = (int64_t)lane * per; c < cols; c += 64 * per * kL) {
            uint4 v[kL];
#pragma unroll
            for (int l = 0; l < kL; ++l) v[l] = ld16_any(p + min(c + (int64_t)l * 64 * per, cols - per) * esz);
            __builtin_amdgcn_sched_barrier(0);  // all loads issue before the first use
#pragma unroll
            for (int l = 0; l < kL; ++l) {
                if (DT == FP8_DT_BF16) mm = fold_bf16(mm, v[l]);
                else m = fold_f32(m, v[l]);
            }
        }
        if (DT == FP8_DT_BF16) m = max((uint32_t)mm.x, (uint32_t)mm.y);
    } else if (lane < cols) {
        m = elem_mag<DT>(p, lane);
    }
    m = wave_max(m);
    if (lane == 0) rmax[r] = m;
}

// One segment [b0, b1) as thread tid of nth, which all call it: the maximum of
// its rows' words, Eq. 3, and the bias over the words.  reduce: the maximum
// over the nth threads.
template <int DT, int FMT, int NTH, typename Reduce>
__device__ __forceinline__ void seg_finish(int64_t seg, int64_t b0, int64_t b1, int tid, int32_t margin,
                                           int32_t* __restrict__ bias, uint32_t* __restrict__ amax,
                                           uint32_t* __restrict__ flags, uint32_t* __restrict__ rowb, Reduce reduce) {
    uint32_t m = 0;
    for (int64_t i = b0 + tid; i < b1; i += 4 * NTH) {
        uint32_t v[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) v[l] = rowb[min(i + l * NTH, b1 - 1)];
        m = max(m, max(max(v[0], v[1]), max(v[2], v[3])));
    }
    m = reduce(m);
    const uint32_t a32 = canon_amax(DT == FP8_DT_BF16 ? m << 16 : m);
    uint32_t fl;
    const int32_t b = bias_of<FMT>(a32, margin, &fl);
    if (tid == 0) {
        bias[seg] = b;
        amax[seg] = a32;
        if (flags) flags[seg] = fl;
    }
    for (int64_t i = b0 + tid; i < b1; i += NTH) rowb[i] = (uint32_t)b;
}

// Maximum over a workgroup of NTH threads; red may be reused after the next barrier.
template <int NTH>
__device__ __forceinline__ uint32_t wg_max(uint32_t m, uint32_t* red) {
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NTH / 64; ++w) m = max(m, red[w]);
    return m;
}

// A workgroup per segment.  Few segments take wide workgroups (long
// segments), more take narrow ones (more of them resident).
template <int DT, int FMT, int kSegThreads>
__global__ __launch_bounds__(kSegThreads) void seg_bias_kernel(const int32_t* __restrict__ off, int64_t rows,
                                                               int32_t margin, int32_t* __restrict__ bias,
                                                               uint32_t* __restrict__ amax, uint32_t* __restrict__ flags,
                                                               uint32_t* __restrict__ rowb) {
    __shared__ uint32_t red[kSegThreads / 64];
    const int64_t b0 = min(max((int64_t)off[blockIdx.x], (int64_t)0), rows);
    const int64_t b1 = min(max((int64_t)off[blockIdx.x + 1], b0), rows);
    seg_finish<DT, FMT, kSegThreads>(blockIdx.x, b0, b1, threadIdx.x, margin, bias, amax, flags, rowb,
                                     [&](uint32_t m) { return wg_max<kSegThreads>(m, red); });
}

// Very many segments (short ones on average): a wave per segment, four at a
// time per workgroup, over a bounded grid; a segment of more than
// kSegWaveRows rows is taken by the whole workgroup.  A workgroup per segment
// spends its time on launching workgroups, and from 2^24 segments on is more
// than one launch holds.
// Up to kSegMany a workgroup per segment is as fast (20000 rows in 4000
// segments: 18.1 us) and takes a long one among short ones with all its waves;
// beyond, 20000 x 64 in 20000: 27.7 -> 20.7 us, 10^6 x 64 in 10^6: 928 -> 528.
constexpr int kSegWaves = 4, kSegWaveRows = 1024, kSegManyBlocks = 16384, kSegMany = 4096;

template <int DT, int FMT>
__global__ __launch_bounds__(64 * kSegWaves) void seg_bias_many_kernel(const int32_t* __restrict__ off, int64_t nseg,
                                                                       int64_t rows, int32_t margin,
                                                                       int32_t* __restrict__ bias,
                                                                       uint32_t* __restrict__ amax,
                                                                       uint32_t* __restrict__ flags,
                                                                       uint32_t* __restrict__ rowb) {
    __shared__ uint32_t red[kSegWaves];
    __shared__ int64_t bound[kSegWaves + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int64_t s0 = (int64_t)blockIdx.x * kSegWaves; s0 < nseg; s0 += (int64_t)gridDim.x * kSegWaves) {
        __syncthreads();  // bound and red are free
        if (threadIdx.x <= kSegWaves)
            bound[threadIdx.x] = min(max((int64_t)off[min(s0 + threadIdx.x, nseg)], (int64_t)0), rows);
        __syncthreads();
        if (s0 + w < nseg && bound[w + 1] - bound[w] <= kSegWaveRows)
            seg_finish<DT, FMT, 64>(s0 + w, bound[w], max(bound[w], bound[w + 1]), lane, margin, bias, amax, flags, rowb,
                                    [](uint32_t m) { return wave_max(m); });
        for (int j = 0; j < kSegWaves && s0 + j < nseg; ++j) {  // the same for every thread
            if (bound[j + 1] - bound[j] <= kSegWaveRows) continue;
            seg_finish<DT, FMT, 64 * kSegWaves>(s0 + j, bound[j], bound[j + 1], threadIdx.x, margin, bias, amax, flags,
                                                rowb, [&](uint32_t m) { return wg_max<64 * kSegWaves>(m, red); });
            __syncthreads();  // red is read
        }
    }
}

template <int DT, int FMT>
__global__ __launch_bounds__(kCastThreads) void cast_rows_kernel(
    const void* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx, const int32_t* __restrict__ rowb,
    uint8_t* __restrict__ q, int64_t ldq, uint8_t* __restrict__ qT, int64_t ldqT, int64_t tiles_c) {
    __shared__ __attribute__((aligned(16))) uint8_t tile[kCastCols * kCastRows];
    cast_tile<DT, FMT, false, true>(x, rows, cols, ldx, 0, q, ldq, qT, ldqT, blockIdx.x / tiles_c,
                                    blockIdx.x % tiles_c, tile, rowb);
}

template <int DT, int FMT>
void launch_quantise_segments_t(const void* x, int64_t rows, int64_t cols, int64_t ldx, int32_t margin,
                                const int32_t* off, int nseg, int32_t* bias, uint32_t* amax, uint32_t* flags,
                                int32_t* rowb, uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT, hipStream_t s) {
    uint32_t* rmax = (uint32_t*)rowb;
    if (rows > 0 && cols > 0)
        hipLaunchKernelGGL((row_max_kernel<DT>), dim3((unsigned)((rows + kRowWaves - 1) / kRowWaves)),
                           dim3(64 * kRowWaves), 0, s, x, rows, cols, ldx, rmax);
    else if (rows > 0)  // rows of no columns: maxima 0
        hipLaunchKernelGGL(fill_words_kernel, dim3((unsigned)std::min<int64_t>((rows + 255) / 256, 1024)), dim3(256), 0, s,
                           rmax, rows, 0u);
    if (nseg <= 64)
        hipLaunchKernelGGL((seg_bias_kernel<DT, FMT, 1024>), dim3((unsigned)nseg), dim3(1024), 0, s, off, rows, margin, bias,
                           amax, flags, rmax);
    else if (nseg > kSegMany)
        hipLaunchKernelGGL((seg_bias_many_kernel<DT, FMT>),
                           dim3((unsigned)std::min<int64_t>(((int64_t)nseg + kSegWaves - 1) / kSegWaves, kSegManyBlocks)),
                           dim3(64 * kSegWaves), 0, s, off, (int64_t)nseg, rows, margin, bias, amax, flags, rmax);
    else
        hipLaunchKernelGGL((seg_bias_kernel<DT, FMT, 256>), dim3((unsigned)nseg), dim3(256), 0, s, off, rows, margin, bias,
                           amax, flags, rmax);
    if (rows > 0 && cols > 0 && (q || qT)) {
        const int64_t tiles_r = (rows + kCastRows - 1) / kCastRows, tiles_c = (cols + kCastCols - 1) / kCastCols;
        hipLaunchKernelGGL((cast_rows_kernel<DT, FMT>), dim3((unsigned)(tiles_r * tiles_c)), dim3(kCastThreads), 0, s,
                           x, rows, cols, ldx, rowb, q, ldq, qT, ldqT, tiles_c);
    }
}

// Statistical mode of n biases (most frequent value; the smallest of equally
// frequent ones), appended to a ring buffer: ring[*count % capacity] = mode,
// then *count += 1.  One workgroup; biases outside [-kModeRange, kModeRange)
// are counted at the nearest end of that range.
constexpr int kModeRange = 1024;

__global__ __launch_bounds__(256) void bias_mode_kernel(const int32_t* __restrict__ b, int64_t n,
                                                        int32_t* __restrict__ ring, int64_t capacity,
                                                        uint32_t* __restrict__ count) {
    __shared__ uint32_t hist[2 * kModeRange];
    __shared__ uint64_t best[256];
    for (int i = threadIdx.x; i < 2 * kModeRange; i += 256) hist[i] = 0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const int v = max(-kModeRange, min(kModeRange - 1, b[i]));
        atomicAdd(&hist[v + kModeRange], 1u);
    }
    __syncthreads();
    // key: count in the high bits, (2 kModeRange - 1 - bin) in the low 11, so
    // that the largest key is the most frequent bin, and among equals the lowest
    uint64_t k = 0;
    for (int i = threadIdx.x; i < 2 * kModeRange; i += 256)
        if (hist[i]) k = max(k, ((uint64_t)hist[i] << 11) | (uint64_t)(2 * kModeRange - 1 - i));
    best[threadIdx.x] = k;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) best[threadIdx.x] = max(best[threadIdx.x], best[threadIdx.x + off]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int bin = 2 * kModeRange - 1 - (int)(best[0] & 0x7FFull);
        const uint32_t c = *count;
        ring[c % (uint64_t)capacity] = bin - kModeRange;
        *count = c + 1;
    }
}

}  // namespace

int amax_blocks(int64_t n) {
    const int64_t per_block = (int64_t)kAmaxThreads * 8 * 4;  // 4 vectors of 8 bf16 per thread
    int64_t nb = (n + per_block - 1) / per_block;
    if (nb < 1) nb = 1;
    if (nb > kAmaxMaxBlocks) nb = kAmaxMaxBlocks;
    return (int)nb;
}

int32_t launch_scale_bias(const void* x, int dt, int64_t n, int fmt, int32_t margin, int32_t* bias,
                          uint32_t* amax_bits, uint32_t* flags, uint32_t* partials, hipStream_t s) {
    // n == 0: no partials; the finalize pass sees an amax of 0.
    const int nb = n > 0 ? amax_blocks(n) : 0;
    if (nb > 0 && dt == FP8_DT_BF16)
        hipLaunchKernelGGL(amax_partial_kernel<FP8_DT_BF16>, dim3(nb), dim3(kAmaxThreads), 0, s, x, n, partials);
    else if (nb > 0)
        hipLaunchKernelGGL(amax_partial_kernel<FP8_DT_F32>, dim3(nb), dim3(kAmaxThreads), 0, s, x, n, partials);
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        hipLaunchKernelGGL((amax_finalize_kernel<decltype(D)::value, decltype(F)::value>), dim3(1), dim3(kAmaxThreads), 0,
                           s, partials, nb, margin, bias, amax_bits, flags);
    });
    return hip_status();
}

int32_t launch_bias_from_amax(const uint32_t* amax_bits, int fmt, int32_t margin, int32_t* bias,
                              uint32_t* flags, hipStream_t s) {
    with_fmt(fmt, [&](auto F) {
        hipLaunchKernelGGL(bias_from_amax_kernel<decltype(F)::value>, dim3(1), dim3(64), 0, s, amax_bits, margin, bias, flags);
    });
    return hip_status();
}

int32_t launch_cast(const void* x, int dt, int64_t rows, int64_t cols, int64_t ldx, int fmt,
                    const int32_t* bias, uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT,
                    hipStream_t s) {
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_cast_t<decltype(D)::value, decltype(F)::value>(x, rows, cols, ldx, bias, q, ldq, qT, ldqT, s);
    });
    return hip_status();
}

int32_t launch_quant_check(const void* x, int dt, int64_t rows, int64_t cols, int64_t ldx, int fmt,
                           int32_t margin, const uint32_t* parts, int nparts, const int32_t* used,
                           int32_t* bias, uint32_t* amax_bits, uint32_t* flags, uint8_t* q, int64_t ldq,
                           uint8_t* qT, int64_t ldqT, hipStream_t s) {
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_quant_check_t<decltype(D)::value, decltype(F)::value>(x, rows, cols, ldx, margin, parts, nparts, used,
                                                                     bias, amax_bits, flags, q, ldq, qT, ldqT, s);
    });
    return hip_status();
}

int32_t launch_quantise_delayed(const void* x, int dt, int64_t rows, int64_t cols, int64_t ldx, int fmt,
                                int32_t margin, int32_t* bias, uint32_t* history, int hlen, uint32_t* count,
                                uint32_t* amax_bits, uint32_t* flags, uint8_t* q, int64_t ldq, uint8_t* qT,
                                int64_t ldqT, uint32_t* ws, hipStream_t s) {
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_quantise_delayed_t<decltype(D)::value, decltype(F)::value>(x, rows, cols, ldx, margin, bias, history,
                                                                          hlen, count, amax_bits, flags, q, ldq, qT,
                                                                          ldqT, ws, s);
    });
    return hip_status();
}

int64_t quantise_ws_words(int64_t rows, int64_t cols) {
    const int64_t tiles = ((rows + kCastRows - 1) / kCastRows) * ((cols + kCastCols - 1) / kCastCols);
    return 1 + tiles;
}

int64_t quantise_tiles_upto(int64_t rows, int64_t cols, int64_t limit) {
    const int64_t tr = (rows + kCastRows - 1) / kCastRows, tc = (cols + kCastCols - 1) / kCastCols;
    if (tr == 0 || tc == 0) return 0;
    if (tr > limit / tc) return -1;
    return tr * tc;
}

int32_t launch_quantise(const void* x, int dt, int64_t rows, int64_t cols, int64_t ldx, int fmt,
                        int32_t margin, const int32_t* bias_pred, int32_t* bias, uint32_t* amax_bits,
                        uint32_t* flags, uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT,
                        uint32_t* ws, hipStream_t s) {
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_quantise_t<decltype(D)::value, decltype(F)::value>(x, rows, cols, ldx, margin, bias_pred, bias, amax_bits,
                                                                  flags, q, ldq, qT, ldqT, ws, s);
    });
    return hip_status();
}

int32_t launch_quantise_batch(int n, const QuantDesc* d, int dt, int fmt, int32_t margin, hipStream_t s) {
    if (n == 1)  // the kernels that take one tensor have no descriptor array to walk
        return launch_quantise(d->x, dt, d->rows, d->cols, d->ldx, fmt, margin, d->pred, d->bias, d->amax, d->flags, d->q,
                               d->ldq, d->qT, d->ldqT, d->ws, s);
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_quantise_batch_t<decltype(D)::value, decltype(F)::value>(n, d, margin, s);
    });
    return hip_status();
}

int32_t launch_quantise_segments(const void* x, int dt, int64_t rows, int64_t cols, int64_t ldx, int fmt,
                                 int32_t margin, const int32_t* offsets, int nseg, int32_t* bias, uint32_t* amax_bits,
                                 uint32_t* flags, int32_t* row_bias, uint8_t* q, int64_t ldq, uint8_t* qT,
                                 int64_t ldqT, hipStream_t s) {
    with_dt_fmt(dt, fmt, [&](auto D, auto F) {
        launch_quantise_segments_t<decltype(D)::value, decltype(F)::value>(
            x, rows, cols, ldx, margin, offsets, nseg, bias, amax_bits, flags, row_bias, q, ldq, qT, ldqT, s);
    });
    return hip_status();
}

int32_t launch_bias_mode(const int32_t* bias, int64_t n, int32_t* ring, int64_t capacity, uint32_t* count,
                         hipStream_t s) {
    hipLaunchKernelGGL(bias_mode_kernel, dim3(1), dim3(256), 0, s, bias, n, ring, capacity, count);
    return hip_status();
}

}  // namespace fp8lin
