// HIP kernels of libuq for MI355X (gfx950).
//
// The aggregation step of Algorithm 1 / Algorithm 2 (Sec. 3.1-3.2) as
// streaming kernels, each bound by HBM bandwidth:
//   k_sumsq      per-row, per-chunk fp64 sums of squares        (norm, pass 1)
//   k_finish     fixed-order reduction of the chunk sums, max    (norm, pass 2)
//                over rows, sqrt -> W
//   k_index      shared scale index from the largest |g| over    (Eq. (11) +
//                the workers at each coordinate                    sharing)
//   k_norm_max   several scales, 2..16 rows: the norm's tile     (norm + the
//                sums and the largest |g| over the rows in one     index's input)
//                read of the gradients
//   k_rowsum     sums of those tile sums
//   k_index_prep the rows' sums, W and the index pass's thresholds
//                and exponent table, once per call
//   k_index_max  the shared index from the maxima's keys
//   k_quantise   Philox draws + stochastic rounding + int8 pack  (Eq. (8)/(12))
//   k_sum        int8 (or 4-/2-bit) code rows -> int32           (all-reduce)
//                sums, optionally with the reconstruction applied  (+ Eq. (9)/(13))
//   k_quant_sum  the quantiser's codes added straight into the   (Eq. (8)/(12) +
//                int32 sums, never stored (+ the reconstruction)   all-reduce)
//   k_index_quant_sum  all of up to 16 rows held at once: the     (Eq. (11) +
//                shared index from their exact maxima, then        sharing, (12),
//                k_quant_sum's codes, sums and reconstruction      sum, (13))
//   k_quant_sum_split  one scale, up to 16 rows: the same with    (Eq. (8),
//                no index; k_quant_sum_waves: few coordinates      sum, (9))
//                of 11 to 16 rows, a tile's rows over four waves
//   k_index_quantise  either with the codes stored, and summed    (the same)
//                and reconstructed as they are stored
//   k_step_small a whole step of few coordinates in one block     (Alg. 1 / 2)
//   k_dequant    int32 (+ index) -> fp32                          (Eq. (9)/(13))
//
// Every per-coordinate result is a pure function of its inputs and the
// coordinate index, so the output is independent of the launch geometry;
// the norm's reduction tree depends only on d (and on which norm pass runs).
#include <atomic>

#include "uq_device.hpp"
#include "uq_launch.hpp"

namespace uq {

// ---------------------------------------------------------------------------
// Norm, pass 1: block (c, m) sums g[m][c*chunk .. min(d, (c+1)*chunk)) squared
// in binary64 (each square exact) and stores the partial in part[m*nchunks+c].
// chunk is a multiple of 1024, so every chunk starts 16-byte aligned.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_sumsq(const float* __restrict__ g, int64_t d, int32_t M,
                                                  int64_t ldg, int64_t chunk, int32_t nchunks,
                                                  double* __restrict__ part)
{
    __shared__ double wave_part[kBlock / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int32_t c = blockIdx.x;
    const int64_t begin = static_cast<int64_t>(c) * chunk;
    const int64_t end = begin + chunk < d ? begin + chunk : d;
    const int64_t nvec = (end - begin) >> 2;
    // grid.y covers the rows (more rows than grid.y: the blocks take them in turn)
    for (int32_t m = blockIdx.y; m < M; m += gridDim.y) {
        const float* row = g + static_cast<int64_t>(m) * ldg;
        const float* v4 = row + begin;
        double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
        int64_t j = threadIdx.x;
        for (; j + 3 * kBlock < nvec; j += 4 * kBlock) {
            const f32x4 a = load_nt(v4 + 4 * j);
            const f32x4 b = load_nt(v4 + 4 * (j + kBlock));
            const f32x4 e = load_nt(v4 + 4 * (j + 2 * kBlock));
            const f32x4 f = load_nt(v4 + 4 * (j + 3 * kBlock));
            acc0 = fma((double)a.x, (double)a.x, acc0); acc1 = fma((double)a.y, (double)a.y, acc1);
            acc2 = fma((double)a.z, (double)a.z, acc2); acc3 = fma((double)a.w, (double)a.w, acc3);
            acc0 = fma((double)b.x, (double)b.x, acc0); acc1 = fma((double)b.y, (double)b.y, acc1);
            acc2 = fma((double)b.z, (double)b.z, acc2); acc3 = fma((double)b.w, (double)b.w, acc3);
            acc0 = fma((double)e.x, (double)e.x, acc0); acc1 = fma((double)e.y, (double)e.y, acc1);
            acc2 = fma((double)e.z, (double)e.z, acc2); acc3 = fma((double)e.w, (double)e.w, acc3);
            acc0 = fma((double)f.x, (double)f.x, acc0); acc1 = fma((double)f.y, (double)f.y, acc1);
            acc2 = fma((double)f.z, (double)f.z, acc2); acc3 = fma((double)f.w, (double)f.w, acc3);
        }
        for (; j < nvec; j += kBlock) {
            const f32x4 a = load_nt(v4 + 4 * j);
            acc0 = fma((double)a.x, (double)a.x, acc0); acc1 = fma((double)a.y, (double)a.y, acc1);
            acc2 = fma((double)a.z, (double)a.z, acc2); acc3 = fma((double)a.w, (double)a.w, acc3);
        }
        // at most three trailing coordinates (only in the last chunk when d % 4 != 0)
        const int64_t tail = begin + (nvec << 2) + threadIdx.x;
        if (tail < end) {
            const double x = row[tail];
            acc0 = fma(x, x, acc0);
        }
        const double s = wave_sum((acc0 + acc1) + (acc2 + acc3));
        if (lane == 0)
            wave_part[wave] = s;
        __syncthreads();
        if (threadIdx.x == 0)
            part[static_cast<int64_t>(m) * nchunks + c] = (wave_part[0] + wave_part[1]) + (wave_part[2] + wave_part[3]);
        __syncthreads();  // wave_part is reused for the next row
    }
}

// ---------------------------------------------------------------------------
// Norm, pass 2 (one block of kFinishThreads): S_m = fixed-order sum of row m's
// chunk partials (lane-strided sequential sums, then a fixed butterfly), one
// wave per row (16 rows at once); W = RN32(sqrt(max_m S_m)), NaN if any S_m
// is NaN.
// ---------------------------------------------------------------------------
constexpr int kFinishThreads = 1024;

__global__ __launch_bounds__(kFinishThreads) void k_finish(const double* __restrict__ part, int32_t nchunks,
                                                           int32_t M, float* __restrict__ w)
{
    __shared__ double wave_best[kFinishThreads / 64];
    __shared__ int wave_nan[kFinishThreads / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    double best = 0.0;
    bool any_nan = false;
    for (int32_t m = wave; m < M; m += kFinishThreads / 64) {
        // nchunks <= 1024: at most 16 partials per lane, all loads in flight at once
        const double* p = part + static_cast<int64_t>(m) * nchunks;
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int32_t c = lane + 64 * j;
            x[j] = c < nchunks ? p[c] : 0.0;
        }
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j)
            s += x[j];
        const double S = wave_sum(s);
        any_nan = any_nan || (S != S);
        best = S > best ? S : best;
    }
    if (lane == 0) {
        wave_best[wave] = best;
        wave_nan[wave] = any_nan ? 1 : 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
        int nan = 0;
        for (int i = 0; i < kFinishThreads / 64; ++i) {
            b = wave_best[i] > b ? wave_best[i] : b;
            nan |= wave_nan[i];
        }
        *w = nan ? __builtin_nanf("") : static_cast<float>(sqrt(b));
    }
}

// ---------------------------------------------------------------------------
// Shared scale index.  The per-worker rule (largest k with
// RN32(|g| inv_k) <= s_0) is non-increasing in |g|, so the minimum over the
// workers is the rule applied to the largest usable |g| at the coordinate;
// a coordinate with no usable |g| (all zero / non-finite) takes K-1.
// Four coordinates per thread per step, float4 loads over the M rows.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t index_of(float amax, const float* inv, int32_t K, float s0,
                                             bool zero)
{
    if (zero || !(amax > 0.0f))
        return static_cast<uint32_t>(K - 1);
    int32_t count = 0;
#pragma unroll
    for (int k = 0; k < kMaxScales; ++k)
        if (k < K)
            count += (amax * inv[k] <= s0) ? 1 : 0;
    return static_cast<uint32_t>(count > 0 ? count - 1 : 0);
}

__device__ __forceinline__ float usable_or_zero(float v)
{
    const float a = fabsf(v);
    return a <= kFloatMax ? a : 0.0f;  // NaN compares false -> 0
}

// Largest usable |g| over the M rows at quad q.
__device__ __forceinline__ f32x4 rows_amax(const float* __restrict__ g, int64_t q, int32_t M, int64_t ldg)
{
    f32x4 amax = {0.0f, 0.0f, 0.0f, 0.0f};
    const float* p = g + (q << 2);
    for (int32_t m = 0; m < M; ++m) {
        const f32x4 v = load_nt(p + static_cast<int64_t>(m) * ldg);
        amax.x = fmaxf(amax.x, usable_or_zero(v.x));
        amax.y = fmaxf(amax.y, usable_or_zero(v.y));
        amax.z = fmaxf(amax.z, usable_or_zero(v.z));
        amax.w = fmaxf(amax.w, usable_or_zero(v.w));
    }
    return amax;
}

// NIB: the index stored as 4-bit fields, two coordinates a byte (the low
// nibble first); a quad's four fields are one 16-bit store.
template <bool NIB>
__global__ __launch_bounds__(kBlock) void k_index(const float* __restrict__ g, int64_t d, int32_t M,
                                                  int64_t ldg, const float* __restrict__ wptr,
                                                  ScaleSet S, uint8_t* __restrict__ idx)
{
    __shared__ float inv_s[kMaxScales];
    const int64_t nquad = d >> 2;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    // the maxima do not need W: the first quad's loads go out before the
    // tables are formed
    f32x4 amax0 = {0.0f, 0.0f, 0.0f, 0.0f};
    if (first < nquad)
        amax0 = rows_amax(g, first, M, ldg);

    const float W = *wptr;
    if (threadIdx.x < S.K)
        inv_s[threadIdx.x] = div_rn32(S.s[threadIdx.x], W);
    __syncthreads();
    float inv[kMaxScales];
#pragma unroll
    for (int k = 0; k < kMaxScales; ++k)
        inv[k] = k < S.K ? __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(
                                 __builtin_bit_cast(int, inv_s[k])))
                         : 0.0f;
    const bool zero = zero_path(W, inv[0]);
    const float s0 = S.s[0];
    const int32_t K = S.K;

    for (int64_t q = first; q < nquad; q += stride) {
        const f32x4 amax = q == first ? amax0 : rows_amax(g, q, M, ldg);
        const int sh = NIB ? 4 : 8;
        const uint32_t packed = index_of(amax.x, inv, K, s0, zero) |
                                (index_of(amax.y, inv, K, s0, zero) << sh) |
                                (index_of(amax.z, inv, K, s0, zero) << (2 * sh)) |
                                (index_of(amax.w, inv, K, s0, zero) << (3 * sh));
        if (NIB)
            *reinterpret_cast<uint16_t*>(idx + (q << 1)) = static_cast<uint16_t>(packed);
        else
            *reinterpret_cast<uint32_t*>(idx + (q << 2)) = packed;
    }
    // trailing d % 4 coordinates (with 4-bit fields one thread forms their
    // bytes, which two coordinates share)
    const int64_t t = (nquad << 2) + static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (blockIdx.x == 0 && t < d && (!NIB || threadIdx.x == 0)) {
        uint32_t nib = 0u;
        for (int64_t i = t; i < (NIB ? d : t + 1); ++i) {
            float amax = 0.0f;
            for (int32_t m = 0; m < M; ++m)
                amax = fmaxf(amax, usable_or_zero(g[static_cast<int64_t>(m) * ldg + i]));
            const uint32_t v = index_of(amax, inv, K, s0, zero);
            if (!NIB) {
                idx[i] = static_cast<uint8_t>(v);
            } else {
                nib |= v << (4 * ((i - t) & 1));
                if (((i - t) & 1) || i + 1 == d) {
                    idx[i >> 1] = static_cast<uint8_t>(nib);
                    nib = 0u;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Fused shared scale for several scales and at most kFuseRows rows: one pass
// over the gradients forms the rows' tile sums of squares and, at every
// coordinate, bits 30..15 of the largest usable |g| over the rows (a key,
// uint16 [d] in the workspace); the index pass then reads the keys
// instead of the M rows, and the rows of the rare coordinates whose key
// equals a threshold's.
//   k_norm_max   block t: tile t of every row (below)
//   k_rowsum     block (b, m) sums partials [b s, (b + 1) s) of row m in a
//                fixed order (s = kRowsumSpan)
//   k_index_prep one block: those sums into S_m (the same order), W (the
//                rule of k_finish), the thresholds, their keys and the
//                exponent table, into the workspace
//   k_index_max  the index of every coordinate from its key and that table
// ---------------------------------------------------------------------------
// Barrier for LDS traffic only: the block's LDS writes are complete and
// visible, while its global loads and stores stay in flight (__syncthreads
// would also wait for those).
__device__ __forceinline__ void sync_lds()
{
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Tile t = the whole quads [256 t, 256 t + 256) (coordinates 1024 t ..) of
// every row; one block per tile, and one more block for the d % 4 trailing
// coordinates, which have a partial of their own (on a grid capped below
// that, blocks stride over the tiles, each tile still with its own partials,
// so the reduction tree does not depend on the grid).  Wave w owns rows
// w, w + 4, ... (ROWS / 4 of them; rows past M re-read row M - 1 and are not
// accumulated): lane l loads quads l, l + 64, l + 128, l + 192 of the tile from
// each of its rows (4 KiB per row per wave), all loads issued at once.  The
// waves' maxima meet in LDS and leave as one coalesced store of their 16-bit
// keys; each row's squares leave as one fp64 partial per tile.  Measured at
// 2^30 coordinates and 16 rows (MI355X), with fp32 maxima then: 12.3 ms
// (0.74 of 8 TB/s) in a probe of this form,
// against 13.8 ms for blocks that loop over 16 tiles with the next tile's
// loads issued before the current tile's store, and 12.8-13.8 ms for every
// looping form tried (double-buffered, no prefetch, 8 waves of 2 rows,
// straight-line runs of 2 to 16 tiles): in them the maxima stores cost about
// 3.7 ms over a pass without them, here 1.3 ms.  The trailing coordinates
// have their own block so that their code adds no registers to the tiles'
// (102 registers with it, four waves per SIMD instead of five).
// The d % 4 trailing coordinates of every row (partial t = ntiles): each
// wave adds its own rows' squares; wave 0 forms the maximum over all rows.
template <int ROWS>
__device__ __forceinline__ void norm_max_tail(const float* __restrict__ g, int64_t d, int32_t M, int64_t ldg,
                                              int64_t ntiles, double* __restrict__ part, uint16_t* __restrict__ keys)
{
    constexpr int RPW = ROWS / 4;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t tail = ((d >> 2) << 2) + lane;
    const int64_t nparts = ntiles + 1;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int m = wave + 4 * r;
        const double x = tail < d ? g[static_cast<int64_t>(m < M ? m : M - 1) * ldg + tail] : 0.0;
        const double sum = wave_sum(x * x);
        if (lane == 0 && m < M)
            part[static_cast<int64_t>(m) * nparts + ntiles] = sum;
    }
    if (wave == 0 && tail < d) {
        float mt = 0.0f;
        for (int32_t m = 0; m < M; ++m)
            mt = fmaxf(mt, usable_or_zero(g[static_cast<int64_t>(m) * ldg + tail]));
        keys[tail] = static_cast<uint16_t>(__builtin_bit_cast(uint32_t, mt) >> 15);
    }
}

// Tile t < ntiles: its maxima's keys and the rows' partials t.
template <int ROWS, bool NT>
__device__ __forceinline__ void norm_max_tile(const float* __restrict__ g, int64_t d, int32_t M, int64_t ldg,
                                              int64_t ntiles, int64_t t, double* __restrict__ part,
                                              uint16_t* __restrict__ keys, f32x4 (*wave_max)[kBlock])
{
    constexpr int RPW = ROWS / 4;  // rows per wave
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t nquad = d >> 2;
    const int64_t q0 = t * kBlock;  // first quad of the tile
    const int64_t qe = q0 + kBlock < nquad ? q0 + kBlock : nquad;  // > q0
    // quads past qe re-read quad qe - 1 (the loads carry no branch) and are
    // zeroed below
    f32x4 v[RPW][4];
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int m = wave + 4 * r;
        const float* row = g + static_cast<int64_t>(m < M ? m : M - 1) * ldg;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t q = q0 + lane + 64 * j;
            v[r][j] = load_nt(row + ((q < qe ? q : qe - 1) << 2));
        }
    }
    f32x4 mx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        mx[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (q0 + lane + 64 * j >= qe) {
#pragma unroll
            for (int r = 0; r < RPW; ++r)
                v[r][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    double acc[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        double a = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a = fma((double)v[r][j].x, (double)v[r][j].x, a);
            a = fma((double)v[r][j].y, (double)v[r][j].y, a);
            a = fma((double)v[r][j].z, (double)v[r][j].z, a);
            a = fma((double)v[r][j].w, (double)v[r][j].w, a);
            mx[j].x = fmaxf(mx[j].x, usable_or_zero(v[r][j].x));
            mx[j].y = fmaxf(mx[j].y, usable_or_zero(v[r][j].y));
            mx[j].z = fmaxf(mx[j].z, usable_or_zero(v[r][j].z));
            mx[j].w = fmaxf(mx[j].w, usable_or_zero(v[r][j].w));
        }
        acc[r] = a;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        wave_max[wave][lane + 64 * j] = mx[j];
    sync_lds();
    const f32x4 m0 = wave_max[0][threadIdx.x], m1 = wave_max[1][threadIdx.x];
    const f32x4 m2 = wave_max[2][threadIdx.x], m3 = wave_max[3][threadIdx.x];
    sync_lds();  // wave_max is reused by the block's next tile
    const int64_t q = q0 + threadIdx.x;
    if (q < qe) {
        f32x4 o;
        o.x = fmaxf(fmaxf(m0.x, m1.x), fmaxf(m2.x, m3.x));
        o.y = fmaxf(fmaxf(m0.y, m1.y), fmaxf(m2.y, m3.y));
        o.z = fmaxf(fmaxf(m0.z, m1.z), fmaxf(m2.z, m3.z));
        o.w = fmaxf(fmaxf(m0.w, m1.w), fmaxf(m2.w, m3.w));
        // the keys: bits 30..15 of the four maxima (exponent and 8 mantissa
        // bits; the sign bit of a maximum is 0), two to a word.
        // __float_as_uint takes the component's value; __builtin_bit_cast of
        // a vector component compiled to a read of component x here.
        u32x2 k;
        k.x = (__float_as_uint(o.x) >> 15) | ((__float_as_uint(o.y) << 1) & 0xFFFF0000u);
        k.y = (__float_as_uint(o.z) >> 15) | ((__float_as_uint(o.w) << 1) & 0xFFFF0000u);
        u32x2* dst = reinterpret_cast<u32x2*>(keys + (q << 2));
        if (NT)
            __builtin_nontemporal_store(k, dst);
        else
            *dst = k;
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const double sum = wave_sum(acc[r]);
        const int m = wave + 4 * r;
        if (lane == 0 && m < M)
            part[static_cast<int64_t>(m) * (ntiles + 1) + t] = sum;
    }
}

// ONE: one block per tile plus the trailing coordinates' block (no loop);
// otherwise blocks stride over them.
template <int ROWS, bool NT, bool ONE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_norm_max(const float* __restrict__ g, int64_t d, int32_t M,
                                                     int64_t ldg, int64_t ntiles, double* __restrict__ part,
                                                     uint16_t* __restrict__ keys)
{
    __shared__ f32x4 wave_max[4][kBlock];
    if (ONE) {
        const int64_t t = blockIdx.x;
        if (t < ntiles)
            norm_max_tile<ROWS, NT>(g, d, M, ldg, ntiles, t, part, keys, wave_max);
        else if (t == ntiles)
            norm_max_tail<ROWS>(g, d, M, ldg, ntiles, part, keys);
        return;
    }
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x)
        norm_max_tile<ROWS, NT>(g, d, M, ldg, ntiles, t, part, keys, wave_max);
    if (blockIdx.x == gridDim.x - 1)
        norm_max_tail<ROWS>(g, d, M, ldg, ntiles, part, keys);
}

// The block's fixed-order sum of p[b0, b1): lane-strided sequential sums
// (16 loads in flight per thread), a fixed butterfly, then the four waves in
// order.  The total is valid in thread 0; wave_part must not be reused before
// the block's next barrier.
__device__ __forceinline__ double rowsum_span(const double* __restrict__ p, int64_t b0, int64_t b1,
                                              double* wave_part)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    double s = 0.0;
    for (int64_t j0 = b0; j0 < b1; j0 += 16 * kBlock) {
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t c = j0 + static_cast<int64_t>(threadIdx.x) + kBlock * j;
            x[j] = c < b1 ? p[c] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j)
            s += x[j];
    }
    s = wave_sum(s);
    if (lane == 0)
        wave_part[wave] = s;
    __syncthreads();
    return (wave_part[0] + wave_part[1]) + (wave_part[2] + wave_part[3]);
}

// Block (b, m) sums part[m][b * span .. min(n, (b + 1) * span)) in the fixed
// order of rowsum_span into out[m * gridDim.x + b].
__global__ __launch_bounds__(kBlock) void k_rowsum(const double* __restrict__ part, int64_t n, int64_t span,
                                                   double* __restrict__ out)
{
    __shared__ double wave_part[kBlock / 64];
    const int64_t b0 = static_cast<int64_t>(blockIdx.x) * span;
    const int64_t b1 = b0 + span < n ? b0 + span : n;
    const double s = rowsum_span(part + static_cast<int64_t>(blockIdx.y) * n, b0, b1, wave_part);
    if (threadIdx.x == 0)
        out[static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x] = s;
}

// k_index_max: a block covers kIndexTile octets of coordinates (4 per
// thread: octets t, t + 256, ..., so each load and store of a wave is
// contiguous), all loaded before the call's constants are read.  The norm
// pass keeps, for each
// coordinate, bits 30..15 of its largest usable |g| over the rows (a key:
// the exponent field and the top 8 mantissa bits; the sign bit is 0).  Keys
// order like the values they truncate.  The per-coordinate rule
// compares thresholds instead of forming products: a -> RN32(a * inv_k) is
// non-decreasing for inv_k > 0, so RN32(a * inv_k) <= s_0 holds exactly for
// a <= T_k, the largest binary32 that passes; k_index_prep finds T_k once
// per call (a few ulp steps from s_0 / inv_k).  A key below T_k's key means a < T_k, a
// key above it a > T_k; only a key equal to T_k's leaves the comparison open,
// and then the coordinate's rows are read again for its exact maximum (at
// the scales used here, about one coordinate in ten thousand).  The count
// #{k : a <= T_k} needs no loop over k when no binade holds two thresholds
// (scales at least about twice apart, as 16^k): every T_k in a higher binade
// than a's counts, none in a lower one, so a table over the 256 values of the
// exponent field gives the count above a's binade and the key of the one
// threshold inside it, and a coordinate costs one lookup and two compares.
// Otherwise the block compares each key with the K thresholds' keys.  The
// thresholds, their keys and the table are formed once per call
// (k_index_prep) rather than in each of the pass's blocks: at 2^30
// coordinates that prologue was most of the pass's VALU work.
constexpr int kIndexOcts = 4;
constexpr int64_t kIndexTile = kIndexOcts * kBlock;
static_assert(kBlock == 256, "the exponent table has one entry per thread");

// Largest binary32 a >= 0 with RN32(a * inv) <= s0, for 0 < inv; 0 when inv
// is infinite (then no positive a passes).
__device__ float index_threshold(float inv, float s0)
{
    if (!(inv <= kFloatMax))
        return 0.0f;
    const double q = static_cast<double>(s0) / static_cast<double>(inv);
    float a = q >= static_cast<double>(kFloatMax) ? kFloatMax : static_cast<float>(q);
    // RN32(q) is within an ulp or two of the boundary; the loops are bounded
    // for safety and take at most a few steps
    for (int i = 0; i < 64 && a > 0.0f && a * inv > s0; ++i)
        a = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) - 1u);
    for (int i = 0; i < 64 && a < kFloatMax; ++i) {
        const float n = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) + 1u);
        if (!(n * inv <= s0))
            break;
        a = n;
    }
    return a;
}

// Scale index of amax from the thresholds: #{k < K : amax <= T_k} - 1 (the
// rule of index_of), K - 1 for a zero amax or on the zero path.
__device__ __forceinline__ uint32_t index_from_count(float amax, int32_t count, int32_t K, bool zero)
{
    if (zero || !(amax > 0.0f))
        return static_cast<uint32_t>(K - 1);
    return static_cast<uint32_t>(count > 0 ? count - 1 : 0);
}

// The index of coordinate i from its exact maximum over the rows (the value
// whose key the norm pass kept); M <= kFuseRows.  Rows past M re-read row
// M - 1 (no change to the maximum), so that the loads carry no branch and
// all are in flight at once.
__device__ __forceinline__ uint32_t index_exact(const float* __restrict__ g, int64_t ldg, int32_t M, int64_t i,
                                             const float* thr, int32_t K)
{
    float v[kFuseRows];
#pragma unroll
    for (int m = 0; m < kFuseRows; ++m)
        v[m] = g[static_cast<int64_t>(m < M ? m : M - 1) * ldg + i];
    float a = 0.0f;
#pragma unroll
    for (int m = 0; m < kFuseRows; ++m)
        a = fmaxf(a, usable_or_zero(v[m]));
    int32_t count = 0;
    for (int k = 0; k < K; ++k)
        count += a <= thr[k] ? 1 : 0;
    return index_from_count(a, count, K, false);
}

// Index of the coordinate with key `key` from the exponent table (entry e:
// the index when the key is not below the limit key of binade e, and that
// key; binades without a threshold hold 0x10000, which every key is below,
// with their index lowered by one); `tie` collects a key equal to the limit's.
__device__ __forceinline__ uint32_t index_from_key(const uint2* tab, uint32_t key, bool& tie)
{
    const uint2 t = tab[key >> 8];
    tie |= key == t.y;
    return t.x + (key < t.y ? 1u : 0u);
}

// The same from the K thresholds' keys (binades that hold two thresholds).
__device__ __forceinline__ uint32_t index_from_keys(const uint32_t* hk, int32_t K, uint32_t key, bool& tie)
{
    int32_t count = 0;
    for (int k = 0; k < K; ++k) {
        count += key < hk[k] ? 1 : 0;
        tie |= key == hk[k];
    }
    return static_cast<uint32_t>(count > 0 ? count - 1 : 0);
}

// Key c of an octet's eight (two per 32-bit word, the lower coordinate in
// the low half).
__device__ __forceinline__ uint32_t octet_key(const u32x4& kv, int c)
{
    const uint32_t w = c < 2 ? kv.x : c < 4 ? kv.y : c < 6 ? kv.z : kv.w;
    return (c & 1) ? w >> 16 : w & 0xFFFFu;
}

// One block: the rows' sums S_m from their kRowsumSpan-partial sums (the
// order of k_rowsum), W = RN32(sqrt(max_m S_m)) (NaN if any S_m is NaN, as
// k_finish), stored to *wptr, then the index pass's constants for the call:
// thresholds T_k, their keys and the exponent table (thread e forms entry e:
// the thresholds in higher binades, every key of binade e being below
// theirs, and the one inside binade e).  On the zero path every coordinate
// gets K - 1.
__global__ __launch_bounds__(kBlock) void k_index_prep(const double* __restrict__ sub, int64_t nsub, int32_t M,
                                                       double* __restrict__ rows, float* __restrict__ wptr,
                                                       ScaleSet S, IndexTables* __restrict__ T)
{
    __shared__ double wave_part[kBlock / 64];
    __shared__ double row_part[kFuseRows][kBlock / 64];
    __shared__ double row_s[kFuseRows];
    __shared__ float thr_s[kMaxScales];
    __shared__ uint32_t hk_s[kMaxScales];
    __shared__ float w_s;
    if (nsub <= kBlock) {
        // at most one partial per thread and row (every d below 2^32): all
        // rows' loads at once, then for each row the arithmetic of
        // rowsum_span (its sequential sum is the one value plus zeros,
        // exactly that value; then the butterfly and the four waves in order)
        const int lane = threadIdx.x & 63;
        const int wave = threadIdx.x >> 6;
        double x[kFuseRows];
#pragma unroll
        for (int m = 0; m < kFuseRows; ++m)
            x[m] = 0.0 + (m < M && threadIdx.x < nsub ? sub[static_cast<int64_t>(m) * nsub + threadIdx.x] : 0.0);
#pragma unroll
        for (int m = 0; m < kFuseRows; ++m) {
            const double s = wave_sum(x[m]);
            if (lane == 0)
                row_part[m][wave] = s;
        }
        __syncthreads();
        if (threadIdx.x < M) {
            const double* w4 = row_part[threadIdx.x];
            const double r = (w4[0] + w4[1]) + (w4[2] + w4[3]);
            rows[threadIdx.x] = r;
            row_s[threadIdx.x] = r;
        }
    } else {
        for (int32_t m = 0; m < M; ++m) {
            const double r = rowsum_span(sub + static_cast<int64_t>(m) * nsub, 0, nsub, wave_part);
            if (threadIdx.x == 0) {
                rows[m] = r;
                row_s[m] = r;
            }
            __syncthreads();  // wave_part is written again by the next row
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double best = 0.0;
        bool any_nan = false;
        for (int32_t m = 0; m < M; ++m) {
            const double r = row_s[m];
            any_nan = any_nan || (r != r);
            best = r > best ? r : best;
        }
        const float W = any_nan ? __builtin_nanf("") : static_cast<float>(sqrt(best));
        *wptr = W;
        w_s = W;
    }
    __syncthreads();
    const float W = w_s;
    const float s0 = S.s[0];
    const int32_t K = S.K;
    const bool zero = zero_path(W, div_rn32(s0, W));
    if (threadIdx.x < K) {
        const float t = zero ? 0.0f : index_threshold(div_rn32(S.s[threadIdx.x], W), s0);
        thr_s[threadIdx.x] = t;
        hk_s[threadIdx.x] = __builtin_bit_cast(uint32_t, t) >> 15;
        T->thr[threadIdx.x] = t;
        T->hk[threadIdx.x] = __builtin_bit_cast(uint32_t, t) >> 15;
    }
    __syncthreads();
    int crowded = 0;
    {
        const uint32_t e = threadIdx.x;
        int32_t above = 0, inside = 0;
        uint32_t kin = 0u;
        for (int k = 0; k < K; ++k) {
            const uint32_t be = __builtin_bit_cast(uint32_t, thr_s[k]) >> 23;
            above += be > e ? 1 : 0;
            if (be == e) {
                ++inside;
                kin = hk_s[k];
            }
        }
        uint2 ent;
        if (zero) {
            ent.x = static_cast<uint32_t>(K - 2);
            ent.y = 0x10000u;
        } else {
            // #{k : a <= T_k} - 1 = above - 1 + [key below kin]; with nothing
            // above, index 0 either way (nor does a tie matter then)
            crowded = inside > 1 ? 1 : 0;
            const bool limit = inside > 0 && above > 0;
            ent.x = static_cast<uint32_t>(above > 0 ? above - 1 : 0) - (limit ? 0u : 1u);
            ent.y = limit ? kin : 0x10000u;
        }
        T->tab[e] = ent;
    }
    const bool by_table = __syncthreads_or(crowded) == 0;
    if (threadIdx.x == 0)
        T->by_table = by_table ? 1 : 0;
}

// NIB: the index stored as 4-bit fields (an octet's eight in one 32-bit
// store), as in k_index.
template <bool NT, bool NIB>
__global__ __launch_bounds__(kBlock) void k_index_max(const uint16_t* __restrict__ keys,
                                                      const float* __restrict__ g, int64_t ldg, int64_t d,
                                                      int32_t M, const IndexTables* __restrict__ T, int32_t K,
                                                      uint8_t* __restrict__ idx)
{
    __shared__ float thr_s[kMaxScales];
    __shared__ uint32_t hk_s[kMaxScales];
    __shared__ uint2 tab_s[256];
    const int64_t noct = d >> 3;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kIndexTile;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kIndexTile;
    u32x4 kv[kIndexOcts];
#pragma unroll
    for (int j = 0; j < kIndexOcts; ++j) {
        const int64_t o = tile0 + threadIdx.x + kBlock * j;
        kv[j] = o < noct ? load_nt(reinterpret_cast<const uint32_t*>(keys + (o << 3))) : u32x4{0u, 0u, 0u, 0u};
    }
    // the call's constants (k_index_prep), through LDS
    tab_s[threadIdx.x] = T->tab[threadIdx.x];
    if (threadIdx.x < K) {
        thr_s[threadIdx.x] = T->thr[threadIdx.x];
        hk_s[threadIdx.x] = T->hk[threadIdx.x];
    }
    const bool by_table = T->by_table != 0;
    __syncthreads();

    for (int64_t t0 = tile0; t0 < noct; t0 += stride) {
        if (t0 != tile0) {
#pragma unroll
            for (int j = 0; j < kIndexOcts; ++j) {
                const int64_t o = t0 + threadIdx.x + kBlock * j;
                kv[j] = o < noct ? load_nt(reinterpret_cast<const uint32_t*>(keys + (o << 3)))
                                 : u32x4{0u, 0u, 0u, 0u};
            }
        }
        uint32_t ties = 0u;  // octets j holding a key equal to a threshold's
        if (by_table) {
#pragma unroll
            for (int j = 0; j < kIndexOcts; ++j) {
                const int64_t o = t0 + threadIdx.x + kBlock * j;
                if (o >= noct)
                    continue;
                const uint32_t k8[8] = {kv[j].x & 0xFFFFu, kv[j].x >> 16, kv[j].y & 0xFFFFu, kv[j].y >> 16,
                                        kv[j].z & 0xFFFFu, kv[j].z >> 16, kv[j].w & 0xFFFFu, kv[j].w >> 16};
                uint32_t ix[8];
                bool tie = false;
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    ix[c] = index_from_key(tab_s, k8[c], tie);
                if (NIB) {
                    const uint32_t packed = ix[0] | (ix[1] << 4) | (ix[2] << 8) | (ix[3] << 12) | (ix[4] << 16) |
                                            (ix[5] << 20) | (ix[6] << 24) | (ix[7] << 28);
                    if (NT)
                        __builtin_nontemporal_store(packed, reinterpret_cast<uint32_t*>(idx + (o << 2)));
                    else
                        *reinterpret_cast<uint32_t*>(idx + (o << 2)) = packed;
                } else {
                    u32x2 packed;
                    packed.x = ix[0] | (ix[1] << 8) | (ix[2] << 16) | (ix[3] << 24);
                    packed.y = ix[4] | (ix[5] << 8) | (ix[6] << 16) | (ix[7] << 24);
                    if (NT)
                        __builtin_nontemporal_store(packed, reinterpret_cast<u32x2*>(idx + (o << 3)));
                    else
                        *reinterpret_cast<u32x2*>(idx + (o << 3)) = packed;
                }
                ties |= tie ? 1u << j : 0u;
            }
        } else {
            // binades holding two thresholds (unusual scale sets): the keys
            // again from memory, one octet at a time
#pragma unroll 1
            for (int j = 0; j < kIndexOcts; ++j) {
                const int64_t o = t0 + threadIdx.x + kBlock * j;
                if (o >= noct)
                    continue;
                const u32x4 kj = load_nt(reinterpret_cast<const uint32_t*>(keys + (o << 3)));
                u32x2 packed = {0u, 0u};
                bool tie = false;
#pragma unroll 1
                for (int c = 0; c < 8; ++c) {
                    const uint32_t v = index_from_keys(hk_s, K, octet_key(kj, c), tie);
                    if (NIB)
                        packed.x |= v << (4 * c);
                    else if (c < 4)
                        packed.x |= v << (8 * c);
                    else
                        packed.y |= v << (8 * (c - 4));
                }
                if (NIB)
                    *reinterpret_cast<uint32_t*>(idx + (o << 2)) = packed.x;
                else
                    *reinterpret_cast<u32x2*>(idx + (o << 3)) = packed;
                ties |= tie ? 1u << j : 0u;
            }
        }
        // keys equal to a threshold's (rare): those coordinates' indices again
        // from their exact maxima, over the index bytes just stored
        while (ties != 0u) {
            const int j = __builtin_ctz(ties);
            ties &= ties - 1u;
            const int64_t o = t0 + threadIdx.x + kBlock * j;
            const u32x4 kj = load_nt(reinterpret_cast<const uint32_t*>(keys + (o << 3)));
            uint32_t word = 0u;  // NIB: the octet's eight fields, stored again whole
#pragma unroll 1
            for (int c = 0; c < 8; ++c) {
                bool tc = false;
                const uint32_t key = octet_key(kj, c);
                uint32_t v = by_table ? index_from_key(tab_s, key, tc) : index_from_keys(hk_s, K, key, tc);
                if (tc)
                    v = index_exact(g, ldg, M, (o << 3) + c, thr_s, K);
                if (NIB)
                    word |= v << (4 * c);
                else if (tc)
                    idx[(o << 3) + c] = static_cast<uint8_t>(v);
            }
            if (NIB)
                *reinterpret_cast<uint32_t*>(idx + (o << 2)) = word;
        }
    }
    // the d % 8 trailing coordinates: threads of block 0 (with 4-bit fields
    // thread 0 alone, since two coordinates share a byte)
    const int64_t t = (noct << 3) + threadIdx.x;
    if (blockIdx.x == 0 && t < d && (!NIB || threadIdx.x == 0)) {
        uint32_t nib = 0u;
        for (int64_t i = t; i < (NIB ? d : t + 1); ++i) {
            bool tie = false;
            const uint32_t key = keys[i];
            uint32_t v = by_table ? index_from_key(tab_s, key, tie) : index_from_keys(hk_s, K, key, tie);
            if (tie)
                v = index_exact(g, ldg, M, i, thr_s, K);
            if (!NIB) {
                idx[i] = static_cast<uint8_t>(v);
            } else {
                nib |= v << (4 * ((i - t) & 1));
                if (((i - t) & 1) || i + 1 == d) {
                    idx[i >> 1] = static_cast<uint8_t>(nib);
                    nib = 0u;
                }
            }
        }
    }
}
// ---------------------------------------------------------------------------
// Quantisation.  One thread handles a group of 8 consecutive coordinates,
// which is exactly one Philox block: its eight 16-bit halves are the high
// halves of the coordinates' uniform words (coordinate j < 4 takes the low
// half of word j, coordinate j >= 4 the high half of word j - 4).  The low
// halves (a second block with counter word 3 = 1) are drawn only when some
// coordinate's high half ties its threshold's (probability 2^-16 each).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t half_of(const uint32_t w[4], int j)
{
    return j < 4 ? (w[j] & 0xFFFFu) : (w[j - 4] >> 16);
}

// Quantise the 8 coordinates v[] of group q of `worker`; returns the codes.
__device__ __forceinline__ void quantise_group(const float v[8], const float inv[8], float s0, uint64_t q,
                                               uint32_t worker, uint32_t key0, uint32_t key1, int32_t code[8])
{
    const uint4 hi = philox4x32_10(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32), worker, 0u,
                                   key0, key1);
    const uint32_t hw[4] = {hi.x, hi.y, hi.z, hi.w};
    float x[8];
    bool tie[8];
    bool any_tie = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        code[j] = quantise_hi(v[j], inv[j], s0, half_of(hw, j), &tie[j], &x[j]);
        any_tie = any_tie || tie[j];
    }
    if (__builtin_expect(any_tie, 0)) {
        const uint4 lo = philox4x32_10(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32), worker, 1u,
                                       key0, key1);
        const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w};
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (tie[j])
                code[j] = quantise_tie(v[j], x[j], half_of(lw, j));
    }
}

// Wave tiles.  A wave quantises 512 consecutive coordinates (64 Philox blocks)
// with perfectly coalesced accesses: lane t holds coordinates 4t..4t+3 ("A")
// and 256+4t..256+4t+3 ("B") of the tile.  The A coordinates of lanes 2u and
// 2u+1 form block 64T+u, their B coordinates block 64T+32+u.  Even lane 2u
// computes block 64T+u, odd lane 2u+1 block 64T+32+u, and the pair swaps the
// 16-bit halves the other needs with one DPP move per word pair.
__device__ __forceinline__ uint32_t swap_pair(uint32_t x)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), 0xB1, 0xF, 0xF, false));
}

// Halves of this lane's A and B coordinates from its own block's words w:
// a01/a23 pack coordinates A0..A3 (coordinate 2k in the low half), b01/b23
// likewise for B.  Even lanes keep the low halves of their own words (their
// A coordinates) and receive the partner's low halves (their B coordinates);
// odd lanes keep high halves (B) and receive the partner's high halves (A).
__device__ __forceinline__ void tile_halves(uint4 w, bool odd, uint32_t* a01, uint32_t* a23, uint32_t* b01,
                                            uint32_t* b23)
{
    const uint32_t sel_lo = 0x05040100u;  // low halves of (src1, src0)
    const uint32_t sel_hi = 0x07060302u;  // high halves of (src1, src0)
    const uint32_t sel_keep = odd ? sel_hi : sel_lo;
    const uint32_t sel_send = odd ? sel_lo : sel_hi;
    const uint32_t keep01 = __builtin_amdgcn_perm(w.y, w.x, sel_keep);
    const uint32_t keep23 = __builtin_amdgcn_perm(w.w, w.z, sel_keep);
    const uint32_t recv01 = swap_pair(__builtin_amdgcn_perm(w.y, w.x, sel_send));
    const uint32_t recv23 = swap_pair(__builtin_amdgcn_perm(w.w, w.z, sel_send));
    *a01 = odd ? recv01 : keep01;
    *a23 = odd ? recv23 : keep23;
    *b01 = odd ? keep01 : recv01;
    *b23 = odd ? keep23 : recv23;
}

// BITS = 8: int8 codes.  BITS = 4 or 2: codes packed low bits first, two or
// four to a byte (every |code| <= s_0 fits the field; checked on the host).
template <int BITS>
__device__ __forceinline__ uint32_t pack_field(const int32_t c[4])
{
    constexpr uint32_t mask = (1u << BITS) - 1u;
    uint32_t w = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        w |= (static_cast<uint32_t>(c[j]) & mask) << (BITS * j);
    return w;
}

// Four consecutive codes (16-bit lanes of p01, p23) in the code row's layout:
// 4, 2 or 1 bytes.
template <int BITS>
__device__ __forceinline__ uint32_t pack_quad(uint32_t p01, uint32_t p23)
{
    const uint32_t w = __builtin_amdgcn_perm(p23, p01, 0x06040200u);
    if (BITS == 8)
        return w;
    if (BITS == 4) {
        const uint32_t x = w & 0x0F0F0F0Fu;
        const uint32_t y = x | (x >> 4);
        return __builtin_amdgcn_perm(0u, y, 0x0C0C0200u);
    }
    const uint32_t x = w & 0x03030303u;
    const uint32_t y = x | (x >> 6);
    return (y | (y >> 12)) & 0xFFu;
}

// Stores a lane's A and B quads of codes of one tile (pairs p[0], p[1] and
// p[2], p[3]) to the tile's bytes of a code row.
template <int BITS, bool NT>
__device__ __forceinline__ void store_quads(uint8_t* tile, const uint32_t p[4])
{
    const uint32_t a = pack_quad<BITS>(p[0], p[1]), b = pack_quad<BITS>(p[2], p[3]);
    const uint32_t at = (threadIdx.x & 63u) * (BITS / 2);
    if (BITS == 8) {
        store_through<NT>(tile, at, a);
        store_through<NT>(tile, at + 256, b);
    } else if (BITS == 4) {
        store_through<NT>(tile, at, static_cast<uint16_t>(a));
        store_through<NT>(tile, at + 128, static_cast<uint16_t>(b));
    } else {
        store_through<NT>(tile, at, static_cast<uint8_t>(a));
        store_through<NT>(tile, at + 64, static_cast<uint8_t>(b));
    }
}

// One tile's inputs for one lane: its A and B gradient quads and, with
// several scales, their four scale indices each.
struct TileIn {
    f32x4 A, B;
    uint32_t ka, kb;
};

// The four 4-bit index fields of a 16-bit word (coordinate 2j in the low
// nibble of byte j) spread to the four bytes of a word, the byte layout.
__device__ __forceinline__ uint32_t nibbles_to_bytes(uint32_t h)
{
    return (h & 0xFu) | ((h << 4) & 0xF00u) | ((h << 8) & 0xF0000u) | ((h << 12) & 0xF000000u);
}

// Index k*_i of the 4-bit layout: the low nibble of byte i / 2 for even i,
// the high nibble for odd i.
__device__ __forceinline__ uint32_t nibble_at(const uint8_t* __restrict__ idx4, int64_t i)
{
    return (static_cast<uint32_t>(idx4[i >> 1]) >> ((i & 1) * 4)) & 0xFu;
}

// NIB: the index is held as 4-bit fields (two coordinates a byte); its
// fields are spread to bytes here, so that everything after the load is the
// byte layout's.
template <bool MULTI, bool NIB = false>
__device__ __forceinline__ TileIn load_tile(const float* __restrict__ row, const uint8_t* __restrict__ idx,
                                            int64_t a_off)
{
    TileIn in;
    in.A = load_nt(row + a_off);
    in.B = load_nt(row + a_off + 256);
    if (MULTI && NIB) {
        in.ka = nibbles_to_bytes(*reinterpret_cast<const uint16_t*>(idx + (a_off >> 1)));
        in.kb = nibbles_to_bytes(*reinterpret_cast<const uint16_t*>(idx + ((a_off + 256) >> 1)));
    } else {
        in.ka = MULTI ? *reinterpret_cast<const uint32_t*>(idx + a_off) : 0u;
        in.kb = MULTI ? *reinterpret_cast<const uint32_t*>(idx + a_off + 256) : 0u;
    }
    return in;
}

// This lane's Philox counter word 0 in tile T (and the tile's word 1): block
// 64 T + u for even lane 2u, 64 T + 32 + u for odd lane 2u + 1.
__device__ __forceinline__ uint32_t tile_c0(int64_t T)
{
    const uint32_t lane = threadIdx.x & 63u;
    return (static_cast<uint32_t>(T) << 6) | (lane >> 1) | ((lane & 1u) << 5);
}
__device__ __forceinline__ uint32_t tile_c1(int64_t T)
{
    return static_cast<uint32_t>(static_cast<uint64_t>(T) >> 26);
}

// |code| of a lane's eight coordinates of one row as four 16-bit lane pairs
// (A0 A1, A2 A3, B0 B1, B2 B3), and sgn their signs (1 or -1 per lane): the
// codes are mag * sgn.  v: the lane's coordinates; inv: their s_k / W, times
// 2^16 when PRE (then s0x = s0 * 2^16).  Every lane of the wave must call it
// (DPP exchange, wave-uniform branches).
//
// With T = floor(x * 2^16) = l * 2^16 + th and a uniform high half r, the
// sum u = T + (2^16 - 1 - r) carries into its upper half exactly when
// r < th, so u >> 16 = l + [r < th]: one add on the complemented half.  Its
// lower half is 2^16 - 1 exactly when r == th, the tie the low halves
// decide.  A lane with a tie, or with a T above s0 * 2^16 (x clamped, or an
// infinite v; NaN converts to 0, which is its code), sends the wave to the
// exact form below; about one tile in 128 does.  Without pre every tile
// goes there.  Against forming level,
// threshold and compare in 16-bit lanes, and the first Philox rounds per
// row, this is 30% fewer VALU issue slots a row.
// Returns whether the wave needs the exact form; h: the complemented high
// halves (A0 A1, A2 A3, B0 B1, B2 B3), kept for it.
__device__ __forceinline__ bool fast_mags(const float v[8], const float inv[8], float s0x, const LaneKey& lk,
                                          const RowKey& rk, uint32_t key0, uint32_t key1, uint32_t h[4],
                                          u16x2 mag[4], u16x2 sgn[4])
{
    const bool odd = (threadIdx.x & 1) != 0;
    tile_halves(philox_tail_not(rk, lk, key0, key1), odd, &h[0], &h[1], &h[2], &h[3]);
    uint32_t T[8], u[8];
    uint32_t t_max = 0u, tie = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        T[j] = cvt_u32_sat(fabsf(v[j]) * inv[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        t_max = max(max(T[2 * j], T[2 * j + 1]), t_max);
        u[2 * j] = add_half<0>(T[2 * j], h[j]);
        u[2 * j + 1] = add_half<1>(T[2 * j + 1], h[j]);
        tie = max3_lo16(tie, u[2 * j], u[2 * j + 1]);
        mag[j] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(u[2 * j + 1], u[2 * j], 0x07060302u));
        sgn[j] = pair_signs(v[2 * j], v[2 * j + 1]);
    }
    return __ballot(t_max > static_cast<uint32_t>(s0x) || static_cast<uint16_t>(tie) == 0xFFFFu) != 0;
}

// The exact magnitudes: the low halves drawn too, from the block of counter
// (c0, c1, worker, 1).
__device__ __forceinline__ void exact_mags(const float v[8], const float inv[8], float s0x, bool pre, uint32_t c0,
                                           uint32_t c1, uint32_t worker, uint32_t key0, uint32_t key1,
                                           const uint32_t h[4], u16x2 mag[4])
{
    const bool odd = (threadIdx.x & 1) != 0;
    uint32_t lo[4];
    tile_halves(philox4x32_10(c0, c1, worker, 1u, key0, key1), odd, &lo[0], &lo[1], &lo[2], &lo[3]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t m0 = exact_magnitude(v[2 * j], inv[2 * j], s0x, pre, ~h[j] & 0xFFFFu, lo[j] & 0xFFFFu);
        const uint32_t m1 = exact_magnitude(v[2 * j + 1], inv[2 * j + 1], s0x, pre, ~h[j] >> 16, lo[j] >> 16);
        mag[j] = u16x2{static_cast<uint16_t>(m0), static_cast<uint16_t>(m1)};
    }
}

// Both for one row.
__device__ __forceinline__ void tile_mags(const float v[8], const float inv[8], float s0x, bool pre, int64_t T,
                                          uint32_t worker, uint32_t key0, uint32_t key1, u16x2 mag[4], u16x2 sgn[4])
{
    const uint32_t c0 = tile_c0(T), c1 = tile_c1(T);
    uint32_t h[4];
    const bool rare = fast_mags(v, inv, s0x, lane_key(c0, 0u, key1), row_key(c1, worker, key0), key0, key1, h, mag, sgn);
    if (__builtin_expect(!pre || rare, 0))
        exact_mags(v, inv, s0x, pre, c0, c1, worker, key0, key1, h, mag);
}

// The call's constants in one wave: lane k < K forms scale k's entries.
struct WaveScale {
    float s0x;       // s_0 * 2^16 when pre, else s_0
    bool pre;
    // lane k's s_k / W, the same times 2^16 when pre, and RN32(W / (M s_k));
    // 0 on the zero path
    float raw, inv, deq;
};

__device__ __forceinline__ float lane_value(float x, int32_t lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// The scales come to their lanes through scalar loads: a vector load of them
// here would be waited for behind the rows' loads, which the counter of
// outstanding loads retires in order, and so would everything formed from
// it (measured on 4 rows of 25.6 M coordinates with four scales: 113.7 us against 108.1; 8 rows of 11.2 M: 79.5 against 73.3).
template <bool MULTI>
__device__ __forceinline__ WaveScale wave_scale(float W, const ScaleSet& S, int32_t M)
{
    WaveScale c;
    float s = S.s[0];
    if (MULTI) {
#pragma unroll
        for (int k = 1; k < kMaxScales; ++k)
            __asm__("v_writelane_b32 %0, %1, %2" : "+v"(s) : "s"(S.s[k]), "n"(k));
    }
    const float q = div_rn32(s, W);
    const float s0 = S.s[0];
    const bool zero = zero_path(W, lane_value(q, 0));
    // the largest entry is the last scale's; 2^16 times it stays finite
    c.pre = zero || lane_value(q, MULTI ? S.K - 1 : 0) <= 0x1p100f;
    c.raw = zero ? 0.0f : q;
    c.inv = c.pre ? c.raw * 65536.0f : c.raw;
    c.s0x = c.pre ? s0 * 65536.0f : s0;
    // M * s_k is exactly representable in binary32 (checked on the host)
    c.deq = zero ? 0.0f : div_rn32(W, static_cast<float>(static_cast<double>(M) * static_cast<double>(s)));
    return c;
}

// One tile's scale entries for one lane: its A and B quads' entries of `inv`
// (LDS, several scales) or the one scale's.
template <bool MULTI>
__device__ __forceinline__ void tile_scales(const TileIn& in, const float* inv_t, float inv0, uint32_t kmax,
                                            float inv[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        inv[j] = MULTI ? inv_t[min((in.ka >> (8 * j)) & 0xFFu, kmax)] : inv0;
        inv[j + 4] = MULTI ? inv_t[min((in.kb >> (8 * j)) & 0xFFu, kmax)] : inv0;
    }
}

// The coordinates of one row past its last whole tile (fewer than 512), in
// groups of 8 contiguous coordinates, one per lane of one wave.  inv_s holds
// s_k / W (not scaled).
template <bool MULTI, int BITS>
__device__ __forceinline__ void quantise_tail(const float* __restrict__ row, uint8_t* __restrict__ out,
                                              const uint8_t* __restrict__ idx, int64_t d, int64_t ntiles,
                                              const float* inv_s, float inv0, float s0, uint32_t kmax,
                                              uint32_t worker, uint32_t key0, uint32_t key1)
{
    const int64_t q = (ntiles << 6) + (threadIdx.x & 63);
    const int64_t base = q << 3;
    if (base >= d)
        return;
    float v[8], inv[8];
    int32_t code[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool in = base + j < d;
        v[j] = in ? row[base + j] : 0.0f;
        inv[j] = MULTI ? inv_s[min(static_cast<uint32_t>(in ? idx[base + j] : 0), kmax)] : inv0;
    }
    quantise_group(v, inv, s0, static_cast<uint64_t>(q), worker, key0, key1, code);
    if (BITS == 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (base + j < d)
                out[base + j] = static_cast<uint8_t>(code[j]);
    } else {
        // the group's 8 codes fill whole bytes of its own (coordinates past d
        // have code 0); the packed row holds them
        if (BITS == 4)
            *reinterpret_cast<uint32_t*>(out + base / 2) = pack_field<4>(code) | (pack_field<4>(code + 4) << 16);
        else
            *reinterpret_cast<uint16_t*>(out + base / 4) =
                static_cast<uint16_t>(pack_field<2>(code) | (pack_field<2>(code + 4) << 8));
    }
}

// The quantiser: MULTI with a per-coordinate scale index, BITS the code
// width (8, or 4 / 2 packed), NT codes stored nontemporally too (launches that
// write more than kThroughNontemporalBytes).  One wave per block and tile
// (x: tiles from tile0, the one past the whole tiles the row's last
// coordinates; y: rows), the tile's loads issued before the tables are formed.
template <bool MULTI, int BITS, bool NT>
__global__ __launch_bounds__(64) void k_quantise(const float* __restrict__ g, int64_t d, int64_t ldg, int32_t worker0,
                                                 const float* __restrict__ wptr, ScaleSet S,
                                                 const uint8_t* __restrict__ idx, uint32_t key0, uint32_t key1,
                                                 int64_t tile0, uint8_t* __restrict__ codes, int64_t ldc)
{
    __shared__ float inv_s[kMaxScales];  // s_k / W
    __shared__ float inv_p[kMaxScales];  // s_k / W * 2^16 when pre
    const int32_t r = blockIdx.y;
    const uint32_t worker = static_cast<uint32_t>(worker0) + static_cast<uint32_t>(r);
    const float* row = g + static_cast<int64_t>(r) * ldg;
    uint8_t* out = codes + static_cast<int64_t>(r) * ldc;
    const int64_t ntiles = d >> 9;
    const int64_t T = tile0 + blockIdx.x;
    const int lane = threadIdx.x;
    TileIn in = {};
    if (T < ntiles)
        in = load_tile<MULTI>(row, idx, (T << 9) + 4 * lane);
    const WaveScale c = wave_scale<MULTI>(*wptr, S, 1);
    const uint32_t kmax = static_cast<uint32_t>(S.K - 1);
    if (MULTI && lane < kMaxScales) {
        inv_s[lane] = c.raw;
        inv_p[lane] = c.inv;
    }
    __syncthreads();
    if (T < ntiles) {
        const float v[8] = {in.A.x, in.A.y, in.A.z, in.A.w, in.B.x, in.B.y, in.B.z, in.B.w};
        float inv[8];
        tile_scales<MULTI>(in, inv_p, lane_value(c.inv, 0), kmax, inv);
        u16x2 mag[4], sgn[4];
        tile_mags(v, inv, c.s0x, c.pre, T, worker, key0, key1, mag, sgn);
        uint32_t p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            p[j] = __builtin_bit_cast(uint32_t, static_cast<u16x2>(mag[j] * sgn[j]));
        store_quads<BITS, NT>(out + T * (64 * BITS), p);
    } else {
        quantise_tail<MULTI, BITS>(row, out, idx, d, ntiles, inv_s, lane_value(c.raw, 0), S.s[0], kmax, worker, key0,
                                   key1);
    }
}

// ---------------------------------------------------------------------------
// Integer sum of the rows' codes (the all-reduce), for int8 codes and for
// codes packed as 4- or 2-bit fields.  A block tile of 4096 coordinates:
// thread t unpacks coordinates 16t .. 16t+15 of the tile from one 16-, 8- or
// 4-byte load per row with signed bit-field extracts, eight rows' loads in
// flight at a time.  The tile's sums are then staged through LDS so that the
// int32 stores (and, when accumulating, the loads of the old sums) are
// coalesced: thread t writes quads t, t+256, t+512 and t+768 of the tile.
// With DEQ (1: one scale, 2: several) the same threads also apply the
// reconstruction to the sums they store, so that they need not be read again.
// ---------------------------------------------------------------------------
constexpr int64_t kSumTile = 4096;

// The reconstruction's inputs when it is fused into the sum.
struct DeqArgs {
    const float* w;
    const uint8_t* idx;  // [d] shared scale index (several scales)
    float* out;
    ScaleSet S;
    int32_t M;
    int32_t nt_sum;      // store the sums nontemporally (large d)
};

// The fused sum stores the int32 sums nontemporally when they exceed this
// many bytes: measured 2% faster steps at ResNet-50 and VGG-16 sizes (0.1 to
// 0.55 GB of sums), 1.7% slower at ResNet-18 size (45 MB).
constexpr int64_t kSumNontemporalBytes = int64_t(64) << 20;


// The 16 BITS-bit fields starting at p (16-byte aligned for BITS = 8, 8-byte
// for 4, 4-byte for 2).
template <int BITS>
__device__ __forceinline__ u32x4 load_fields(const uint8_t* p)
{
    u32x4 w = {0u, 0u, 0u, 0u};
    if (BITS == 8) {
        w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    } else if (BITS == 4) {
        const u32x2 h = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
        w.x = h.x;
        w.y = h.y;
    } else {
        w.x = load_nt_u32(p);
    }
    return w;
}

template <int BITS>
__device__ __forceinline__ void add_fields(u32x4 w, int32_t acc[16])
{
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int k = (j * BITS) / 32;
        const uint32_t word = k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
        acc[j] += __builtin_amdgcn_sbfe(static_cast<int32_t>(word), (j * BITS) % 32, BITS);
    }
}

template <int BITS, int DEQ>
__global__ __launch_bounds__(kBlock) void k_sum(const uint8_t* __restrict__ codes, int64_t d, int32_t rows,
                                                int64_t ldc, int32_t accumulate, int32_t* __restrict__ sum,
                                                DeqArgs da)
{
    constexpr int kRowsInFlight = 8;
    // the tile's sums with one padding word after every 16, so that both the
    // row-of-16 writes and the quad reads are free of bank conflicts
    __shared__ int32_t stage[kSumTile + kSumTile / 16];
    __shared__ float deq_s[kMaxScales];
    const int t = threadIdx.x;
    if (DEQ) {
        // deq_k = RN32(W / (M s_k)) as in k_dequant; the barrier after the
        // first tile's staging publishes them
        const float W = *da.w;
        const bool zero = zero_path(W, div_rn32(da.S.s[0], W));
        if (t < da.S.K) {
            const float denom = static_cast<float>(static_cast<double>(da.M) * static_cast<double>(da.S.s[t]));
            deq_s[t] = zero ? 0.0f : div_rn32(W, denom);
        }
    }
    const int32_t kmax = da.S.K - 1;
    for (int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kSumTile; tile0 < d;
         tile0 += static_cast<int64_t>(gridDim.x) * kSumTile) {
        // several scales: the index words of the thread's four quads
        uint32_t kq[4] = {0u, 0u, 0u, 0u};
        if (DEQ == 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t q0 = tile0 + 1024 * c + 4 * t;
                if (q0 + 4 <= d)
                    kq[c] = *reinterpret_cast<const uint32_t*>(da.idx + q0);
            }
        }
        const int64_t c0 = tile0 + 16 * t;
        int32_t acc[16];
#pragma unroll
        for (int j = 0; j < 16; ++j)
            acc[j] = 0;
        if (c0 < d) {
            // fields past d in the last group are read (they lie inside the
            // row's ldc bytes) and dropped below
            const uint8_t* p = codes + c0 * BITS / 8;
            int32_t r = 0;
            for (; r + kRowsInFlight <= rows; r += kRowsInFlight) {
                u32x4 w[kRowsInFlight];
#pragma unroll
                for (int u = 0; u < kRowsInFlight; ++u)
                    w[u] = load_fields<BITS>(p + static_cast<int64_t>(r + u) * ldc);
#pragma unroll
                for (int u = 0; u < kRowsInFlight; ++u)
                    add_fields<BITS>(w[u], acc);
            }
            for (; r < rows; ++r)
                add_fields<BITS>(load_fields<BITS>(p + static_cast<int64_t>(r) * ldc), acc);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j)
            stage[17 * t + j] = acc[j];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int L = 1024 * c + 4 * t;  // tile coordinate of the quad
            const int S = L + (L >> 4);      // its padded LDS index
            const int64_t q0 = tile0 + L;
            if (q0 + 4 <= d) {
                int4 a = make_int4(stage[S], stage[S + 1], stage[S + 2], stage[S + 3]);
                if (accumulate) {
                    const int4 o = *reinterpret_cast<const int4*>(sum + q0);
                    a.x += o.x; a.y += o.y; a.z += o.z; a.w += o.w;
                }
                if (DEQ && da.nt_sum)
                    __builtin_nontemporal_store(i32x4{a.x, a.y, a.z, a.w}, reinterpret_cast<i32x4*>(sum + q0));
                else
                    *reinterpret_cast<int4*>(sum + q0) = a;
                if (DEQ) {
                    f32x4 o;
                    if (DEQ == 2) {
                        const uint32_t kk = kq[c];
                        o.x = static_cast<float>(a.x) * deq_s[min(static_cast<int32_t>(kk & 0xFFu), kmax)];
                        o.y = static_cast<float>(a.y) * deq_s[min(static_cast<int32_t>((kk >> 8) & 0xFFu), kmax)];
                        o.z = static_cast<float>(a.z) * deq_s[min(static_cast<int32_t>((kk >> 16) & 0xFFu), kmax)];
                        o.w = static_cast<float>(a.w) * deq_s[min(static_cast<int32_t>(kk >> 24), kmax)];
                    } else {
                        const float f = deq_s[0];
                        o.x = static_cast<float>(a.x) * f;
                        o.y = static_cast<float>(a.y) * f;
                        o.z = static_cast<float>(a.z) * f;
                        o.w = static_cast<float>(a.w) * f;
                    }
                    store_nt(da.out + q0, o);
                }
            } else {
                for (int j = 0; j < 4 && q0 + j < d; ++j) {
                    const int32_t v = stage[S + j] + (accumulate ? sum[q0 + j] : 0);
                    sum[q0 + j] = v;
                    if (DEQ) {
                        const int32_t k = DEQ == 2 ? min(static_cast<int32_t>(da.idx[q0 + j]), kmax) : 0;
                        da.out[q0 + j] = static_cast<float>(v) * deq_s[k];
                    }
                }
            }
        }
        __syncthreads();  // the next tile reuses stage
    }
}

// ---------------------------------------------------------------------------
// Reconstruction: out_i = RN32(sum_i * deq_k), deq_k = RN32(W / (M s_k)).
// ---------------------------------------------------------------------------
// One wave per block; a lane takes one quad with one scale, two (256
// coordinates apart) with several, where the index lookups then overlap (one
// quad and two, 138 M coordinates: one scale 164 and 175 us, four scales 195
// and 178; 25.6 M: 31.5 and 33.7, 38.0 and 34.6).  NT: the outputs leave
// nontemporally, beyond kSumNontemporalBytes of them as the sums do: one
// rank's calls at 25.6 M coordinates (102 MB of outputs) 78.1 us written
// through, 75.2 nontemporal.
constexpr int dequant_quads(bool multi)
{
    return multi ? 2 : 1;
}

template <bool MULTI, bool NT>
__global__ __launch_bounds__(64) void k_dequant(const int32_t* __restrict__ sum, int64_t d, int32_t M,
                                                const float* __restrict__ wptr, ScaleSet S,
                                                const uint8_t* __restrict__ idx, int64_t tile0,
                                                float* __restrict__ out)
{
    __shared__ float deq_s[kMaxScales];
    const int lane = threadIdx.x;
    const int64_t T = tile0 + blockIdx.x;
    constexpr int kQuads = dequant_quads(MULTI);
    const int64_t t_off = T * (256 * kQuads);
    const bool whole = T < d / (256 * kQuads);
    i32x4 s[kQuads] = {};
    uint32_t kk[kQuads] = {};
    if (whole) {
#pragma unroll
        for (int h = 0; h < kQuads; ++h) {
            const int64_t i = t_off + 256 * h + 4 * lane;
            s[h] = load_nt(sum + i);
            if (MULTI)
                kk[h] = *reinterpret_cast<const uint32_t*>(idx + i);
        }
    }
    const WaveScale c = wave_scale<MULTI>(*wptr, S, M);
    const float deq0 = lane_value(c.deq, 0);
    const uint32_t kmax = static_cast<uint32_t>(S.K - 1);
    if (MULTI && lane < kMaxScales)
        deq_s[lane] = c.deq;
    __syncthreads();
    if (whole) {
#pragma unroll
        for (int h = 0; h < kQuads; ++h) {
            const auto f = [&](int j) { return MULTI ? deq_s[min((kk[h] >> (8 * j)) & 0xFFu, kmax)] : deq0; };
            f32x4 o;
            o.x = static_cast<float>(s[h].x) * f(0);
            o.y = static_cast<float>(s[h].y) * f(1);
            o.z = static_cast<float>(s[h].z) * f(2);
            o.w = static_cast<float>(s[h].w) * f(3);
            if (NT)
                store_nt(out + t_off + 256 * h + 4 * lane, o);
            else
                store_through<false>(out + t_off, 1024 * h + 16 * lane, o);
        }
    } else {
        for (int64_t i = t_off + lane; i < d; i += 64)
            out[i] = static_cast<float>(sum[i]) * (MULTI ? deq_s[min(static_cast<uint32_t>(idx[i]), kmax)] : deq0);
    }
}

// ---------------------------------------------------------------------------
// Quantise and sum in one pass (Eq. (8)/(12) and the all-reduce of Algorithm
// 1/2): the rows' codes, exactly those k_quantise would store, are added into
// the int32 sums in registers and never stored.  A wave takes one
// 512-coordinate tile (the lane layout of k_quantise: quads A = 4t .. 4t+3
// and B = 256+4t .. 256+4t+3) of every row in turn, so the shared index and
// the tables are looked up once per tile; the next row's loads go out before
// the current row is coded.  The tile's sums are then stored once (the old
// sums added first when accumulating) and, with DEQ, so is the reconstruction
// of those sums, RN32(sum * deq_k).  Per streamed row this moves 4 + 1 bytes
// in and 4 (+ 4 read when accumulating) per coordinate, against 6 + 9 for the
// quantiser followed by the sum.
// ---------------------------------------------------------------------------

// The codes of up to kPairRows rows are summed in the 16-bit lanes of the
// pair registers (|sum| <= 256 * 127 < 2^15, so the wrapped 16-bit sums are
// exact), then widened to int32.
constexpr int32_t kPairRows = 256;

template <bool NT>
__device__ __forceinline__ i32x4 load_sum4(const int32_t* p)
{
    if (NT)
        return __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(p));
    return *reinterpret_cast<const i32x4*>(p);
}

// Adds the 16-bit lane sums of h[4] (codes A0 A1, A2 A3, B0 B1, B2 B3) to the
// int32 sums acc[8] and clears h.
__device__ __forceinline__ void widen_pairs(uint32_t h[4], int32_t acc[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        acc[2 * j] += __builtin_amdgcn_sbfe(static_cast<int32_t>(h[j]), 0, 16);
        acc[2 * j + 1] += __builtin_amdgcn_sbfe(static_cast<int32_t>(h[j]), 16, 16);
        h[j] = 0u;
    }
}

// The coordinates past the last whole tile (fewer than 512): lane t of one
// wave takes the 8 contiguous coordinates of group ntiles * 64 + t for every
// row, then stores their sums (and reconstruction).  inv_s holds s_k / W (not
// scaled).  NIB as for load_tile.
template <bool MULTI, bool ACC, bool DEQ, bool NIB = false>
__device__ __forceinline__ void quant_sum_tail(const float* __restrict__ g, int64_t d, int64_t ldg, int32_t rows,
                                               uint32_t worker0, const uint8_t* __restrict__ idx, int64_t ntiles,
                                               const float* inv_s, float inv0, float s0, uint32_t kmax,
                                               uint32_t key0, uint32_t key1, int32_t* __restrict__ sum,
                                               const float* deq_t, float* __restrict__ out)
{
    const int64_t q = (ntiles << 6) + (threadIdx.x & 63);
    const int64_t base = q << 3;
    if (base >= d)
        return;
    float inv[8];
    uint32_t kk[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t raw = base + j < d ? (NIB ? nibble_at(idx, base + j) : static_cast<uint32_t>(idx[base + j])) : 0u;
        kk[j] = MULTI ? min(raw, kmax) : 0u;
        inv[j] = MULTI ? inv_s[kk[j]] : inv0;
    }
    int32_t acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int32_t r = 0; r < rows; ++r) {
        const float* row = g + static_cast<int64_t>(r) * ldg;
        float v[8];
        int32_t code[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = base + j < d ? row[base + j] : 0.0f;
        quantise_group(v, inv, s0, static_cast<uint64_t>(q), worker0 + static_cast<uint32_t>(r), key0, key1, code);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc[j] += code[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (base + j < d) {
            const int32_t s = acc[j] + (ACC ? sum[base + j] : 0);
            sum[base + j] = s;
            if (DEQ)
                out[base + j] = static_cast<float>(s) * deq_t[kk[j]];
        }
    }
}

// How the sums and outputs of a rows pass, or of the one-row form of
// k_quant_sum (kStorePlain: its sums into the L2s), are stored (and, unless
// kStoreThrough, codes nontemporally): through the caches, nontemporally,
// both, or the sums through and the outputs nontemporally.  Steps in a loop
// over three sets of buffers, 8 rows, one scale: 11.2 M coordinates (45 MB of
// sums) 128.4 us through, 129.2 with only the sums through, 132.3
// nontemporal; 12.5 M 147.7, 143.5 and 146.5; 16.0 M 190.0, 184.1 and 188.9;
// 20.0 M sums through 228.0, nontemporal 234.5; 25.6 M 301.4 and 295.9.  Four
// scales (kStoreThrough there stores the outputs nontemporally): 11.2 M 131.3
// sums through, 134.8 nontemporal; 25.6 M (102 MB) 297.5 through, 292.9
// nontemporal, 293.2 both.  A pass of 16 rows of VGG-16 size without work
// (553 MB): 1.72 ms through, 1.68 nontemporal, 1.64 both.
constexpr int kStoreThrough = 0, kStoreNontemporal = 1, kStoreBoth = 2, kStoreSumsThrough = 3,
              kStorePlain = 4;

// ROW1: the one-row form (a streamed worker), compiled apart so that it does
// not carry the row loop's registers.  NIB: the index as 4-bit fields.  NT:
// the old sums loaded, and the sums and outputs stored, nontemporally too.
// One wave per block and tile; tile d >> 9 holds the last coordinates.
template <bool MULTI, bool ACC, bool DEQ, bool NT, bool ROW1, bool NIB>
__global__ __launch_bounds__(64) void k_quant_sum(const float* __restrict__ g, int64_t d, int32_t rows, int64_t ldg,
                                                  int32_t worker0, const float* __restrict__ wptr, ScaleSet S,
                                                  const uint8_t* __restrict__ idx, uint32_t key0, uint32_t key1,
                                                  int64_t tile0, int32_t* __restrict__ sum, int32_t M,
                                                  float* __restrict__ out, int32_t stores)
{
    __shared__ float inv_s[kMaxScales];  // s_k / W
    __shared__ float inv_p[kMaxScales];  // s_k / W * 2^16 when pre
    __shared__ float deq_s[kMaxScales];  // RN32(W / (M s_k))
    const int lane = threadIdx.x;
    const int64_t ntiles = d >> 9;
    const int64_t T = tile0 + blockIdx.x;
    const int64_t t_off = T << 9;
    const int64_t a_off = t_off + 4 * lane;
    const uint32_t w0 = static_cast<uint32_t>(worker0);

    // the tile's loads (row 0, its index words, the old sums) go out before
    // W is read and the tables are formed
    TileIn in = {};
    i32x4 sa = {0, 0, 0, 0}, sb = {0, 0, 0, 0};
    if (T < ntiles) {
        in = load_tile<MULTI, NIB>(g, idx, a_off);
        if (ACC) {
            sa = load_sum4<NT>(sum + a_off);
            sb = load_sum4<NT>(sum + a_off + 256);
        }
    }
    const WaveScale c = wave_scale<MULTI>(*wptr, S, M);
    const uint32_t kmax = static_cast<uint32_t>(S.K - 1);
    const float inv0 = lane_value(c.inv, 0), raw0 = lane_value(c.raw, 0), deq0 = DEQ ? lane_value(c.deq, 0) : 0.0f;
    if (lane < kMaxScales) {
        inv_s[lane] = c.raw;
        inv_p[lane] = c.inv;
        if (DEQ)
            deq_s[lane] = c.deq;
    }
    __syncthreads();
    if (T >= ntiles) {
        quant_sum_tail<MULTI, ACC, DEQ, NIB>(g, d, ldg, rows, w0, idx, ntiles, inv_s, raw0, S.s[0], kmax, key0, key1,
                                             sum, deq_s, out);
        return;
    }
    float inv[8];
    tile_scales<MULTI>(in, inv_p, inv0, kmax, inv);
    int32_t acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t h[4] = {0u, 0u, 0u, 0u};
    int32_t pending = 0;
    f32x4 A = in.A, B = in.B;
    const int32_t nrows = ROW1 ? 1 : rows;
    for (int32_t r = 0; r < nrows; ++r) {
        f32x4 nA = A, nB = B;
        if (!ROW1 && r + 1 < nrows) {
            const float* nrow = g + static_cast<int64_t>(r + 1) * ldg;
            nA = load_nt(nrow + a_off);
            nB = load_nt(nrow + a_off + 256);
        }
        const float v[8] = {A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w};
        u16x2 mag[4], sgn[4];
        tile_mags(v, inv, c.s0x, c.pre, T, w0 + static_cast<uint32_t>(r), key0, key1, mag, sgn);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            h[j] = __builtin_bit_cast(uint32_t, static_cast<u16x2>(mag[j] * sgn[j] + __builtin_bit_cast(u16x2, h[j])));
        if (++pending == kPairRows) {
            widen_pairs(h, acc);
            pending = 0;
        }
        A = nA;
        B = nB;
    }
    widen_pairs(h, acc);
    sa += i32x4{acc[0], acc[1], acc[2], acc[3]};
    sb += i32x4{acc[4], acc[5], acc[6], acc[7]};
    if (ROW1 && !NT && stores == kStorePlain) {
        *reinterpret_cast<i32x4*>(sum + a_off) = sa;
        *reinterpret_cast<i32x4*>(sum + a_off + 256) = sb;
    } else {
        store_through<NT>(sum + t_off, 16 * lane, sa);
        store_through<NT>(sum + t_off, 16 * lane + 1024, sb);
    }
    if (DEQ) {
        // the index words again (two registers live instead of eight indices)
        const auto f = [&](uint32_t word, int j) { return MULTI ? deq_s[min((word >> (8 * j)) & 0xFFu, kmax)] : deq0; };
        f32x4 oa, ob;
        oa.x = static_cast<float>(sa.x) * f(in.ka, 0);
        oa.y = static_cast<float>(sa.y) * f(in.ka, 1);
        oa.z = static_cast<float>(sa.z) * f(in.ka, 2);
        oa.w = static_cast<float>(sa.w) * f(in.ka, 3);
        ob.x = static_cast<float>(sb.x) * f(in.kb, 0);
        ob.y = static_cast<float>(sb.y) * f(in.kb, 1);
        ob.z = static_cast<float>(sb.z) * f(in.kb, 2);
        ob.w = static_cast<float>(sb.w) * f(in.kb, 3);
        if (ROW1 && !NT && stores == kStoreSumsThrough) {
            store_nt(out + a_off, oa);
            store_nt(out + a_off + 256, ob);
        } else {
            store_through<NT>(out + t_off, 16 * lane, oa);
            store_through<NT>(out + t_off, 16 * lane + 1024, ob);
        }
    }
}

// max(m, |x|, |y|) in one instruction (v_maximum3_f32, the absolute values
// by source modifiers).  This maximum propagates NaN: the result is NaN if
// any operand is, else infinite if any operand is, else the largest finite
// value, so a running maximum that stays finite saw finite values only.
__device__ __forceinline__ float max3_abs(float m, float x, float y)
{
    return __builtin_elementwise_maximum(m, __builtin_elementwise_maximum(fabsf(x), fabsf(y)));
}

// ---------------------------------------------------------------------------
// All of up to kFuseRows resident rows quantised, summed and reconstructed in
// one call (one scale, or several with the shared index formed here).  One
// wave per block and 256-coordinate tile: lane t holds quad 4t .. 4t + 3 of
// every row (ROWS, the row count rounded up to even; a row past the last
// re-reads it and is not counted), all loads issued before W is read.  Rows
// are coded two at a time: the lanes of a pair share the Philox block of their
// eight coordinates, so even lanes compute it for row 2p and odd lanes for row
// 2p + 1, and tile_halves' exchange hands each lane its halves for both rows
// (its "A" quad is row 2p's, its "B" quad row 2p + 1's).
//
// What bounds it is the memory system, and the launch shape decides how well
// it streams: with sixteen rows of VGG-16 size, reading them and storing two
// words per coordinate without any work took 1.86 ms with four-wave blocks
// and nontemporal stores, 1.61 ms with one-wave blocks, and 1.59 ms with
// those and write-through stores (1.25 ms for the reads alone).  One quad per
// lane and row keeps 16 rows in 64 registers of 157 to 167 in all
// (UQ_ROWS_WAVES: how many waves share a SIMD).  The tables are formed by the
// wave's first K lanes and kept in LDS; a one-wave block has no barrier to
// wait at.
// ---------------------------------------------------------------------------
struct RowTables {
    float inv[kMaxScales];  // s_k / W, times 2^16 when pre
    float deq[kMaxScales];  // RN32(W / (M s_k))
    RowKey key[kFuseRows];  // each row's part of its Philox blocks
};

// The shared index of a lane's four coordinates from the largest usable |g|
// over the ROWS rows it holds: two rows per instruction with the NaN- and
// infinity-propagating maximum; a result that is not finite means some value
// was not usable (infinite or NaN), and then the lane forms the largest
// usable |g| value by value.  Then the rule itself, #{k : a s_k / W <= s_0}
// - 1, the table's entries broadcast from their lanes.  Written as "not
// above", it also gives K - 1 for a = 0 (0 times an infinite entry is not
// above) and on the zero path (every entry 0).  Against comparing a with
// each scale's threshold this is one multiply more per scale and coordinate
// and saves forming the thresholds in every wave.
template <int ROWS>
__device__ __forceinline__ void quad_index(const f32x4 (&A)[ROWS], const WaveScale& c, int32_t K, uint32_t k[4])
{
    static_assert(ROWS % 2 == 0, "rows are taken in pairs");
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < ROWS; r += 2) {
        a[0] = max3_abs(a[0], A[r].x, A[r + 1].x);
        a[1] = max3_abs(a[1], A[r].y, A[r + 1].y);
        a[2] = max3_abs(a[2], A[r].z, A[r + 1].z);
        a[3] = max3_abs(a[3], A[r].w, A[r + 1].w);
    }
    const uint32_t worst = max(max(__float_as_uint(a[0]), __float_as_uint(a[1])),
                               max(__float_as_uint(a[2]), __float_as_uint(a[3])));
    if (__builtin_expect(worst >= 0x7F800000u, 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            a[j] = 0.0f;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            a[0] = fmaxf(a[0], usable_or_zero(A[r].x));
            a[1] = fmaxf(a[1], usable_or_zero(A[r].y));
            a[2] = fmaxf(a[2], usable_or_zero(A[r].z));
            a[3] = fmaxf(a[3], usable_or_zero(A[r].w));
        }
    }
    uint32_t count[4] = {0u, 0u, 0u, 0u};
    for (int32_t q = 0; q < K; ++q) {
        const float inv = lane_value(c.inv, q);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            count[j] += !(a[j] * inv > c.s0x) ? 1u : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        k[j] = __builtin_elementwise_sub_sat(count[j], 1u);
}

// Loads quad 4t .. 4t + 3 of tile T of every row; with TAIL only the
// coordinates below d, zeros past them.
template <int ROWS, bool TAIL>
__device__ __forceinline__ void load_quads(const float* __restrict__ g, int64_t ldg, int32_t rows, int64_t T,
                                           int64_t d, f32x4 (&A)[ROWS])
{
    const int lane = threadIdx.x & 63;
    const float* tile = g + (T << 8);
    const int64_t left = TAIL ? d - (T << 8) - 4 * lane : 4;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const float* p = tile + static_cast<int64_t>(r < rows ? r : rows - 1) * ldg + 4 * lane;
        if (left >= 4) {
            A[r] = load_nt(p);
        } else {
            A[r].x = left > 0 ? p[0] : 0.0f;
            A[r].y = left > 1 ? p[1] : 0.0f;
            A[r].z = left > 2 ? p[2] : 0.0f;
            A[r].w = 0.0f;
        }
    }
}

// Philox counter words 0 and 1 of this lane in 256-coordinate tile T.
__device__ __forceinline__ uint32_t quad_c0(int64_t T)
{
    return (static_cast<uint32_t>(T) << 5) | ((threadIdx.x & 63u) >> 1);
}
__device__ __forceinline__ uint32_t quad_c1(int64_t T)
{
    return static_cast<uint32_t>(static_cast<uint64_t>(T) >> 27);
}

// Adds mag * sgn of rows 2p ([0], [1]) and, unless it is past the last row,
// 2p + 1 ([2], [3]) to the quad's sums.
__device__ __forceinline__ void add_pair(const u16x2 mag[4], const u16x2 sgn[4], bool both, u16x2& h0, u16x2& h1)
{
    h0 = mag[0] * sgn[0] + h0;
    h1 = mag[1] * sgn[1] + h1;
    if (both) {
        h0 = mag[2] * sgn[2] + h0;
        h1 = mag[3] * sgn[3] + h1;
    }
}

// Stores a lane's four index bytes of tile T (those below d with TAIL).
template <bool TAIL>
__device__ __forceinline__ void store_index(uint8_t* __restrict__ idx, int64_t T, int64_t d, const uint32_t k[4])
{
    const int lane = threadIdx.x & 63;
    const int64_t a_off = T << 8;
    const int64_t left = TAIL ? d - a_off - 4 * lane : 4;
    const uint32_t word = k[0] | (k[1] << 8) | (k[2] << 16) | (k[3] << 24);
    if (left >= 4) {
        store_through<false>(idx + a_off, 4 * lane, word);
    } else {
        for (int j = 0; j < left; ++j)
            idx[a_off + 4 * lane + j] = static_cast<uint8_t>(word >> (8 * j));
    }
}

// The codes of every row pair of tile T: use(p, mag, sgn, nullptr) for each
// pair p as the fast form gives it, then use(p, exact, sgn, fast) for the
// pairs that need the exact form, with what the first call was given.
template <int ROWS, bool TAIL, typename F>
__device__ __forceinline__ void for_row_pairs(const f32x4 (&A)[ROWS], const float* __restrict__ g, int64_t ldg,
                                              int32_t rows, uint32_t worker0, int64_t T, int64_t d,
                                              const WaveScale& c, const float inv[4], const RowTables& tab,
                                              uint32_t key0, uint32_t key1, F use)
{
    const uint32_t c0 = quad_c0(T), c1 = quad_c1(T);
    const uint32_t odd = threadIdx.x & 1u;
    const LaneKey lk = lane_key(c0, 0u, key1);
    const float inv8[8] = {inv[0], inv[1], inv[2], inv[3], inv[0], inv[1], inv[2], inv[3]};
    u16x2 mag[4] = {}, sgn[4];
    uint32_t bits[4];
    uint32_t redo = 0u;  // row pairs that need the exact form (wave-uniform)
#pragma unroll
    for (int p = 0; p < ROWS / 2; ++p) {
        if (2 * p < rows) {
            // the pair's row keys are read when its turn comes (the index
            // depends on the pair before): read ahead for every pair, they
            // take 8 registers each and cost waves on the SIMD (8 rows at
            // 11.2 M coordinates, four scales: 78.7 us against 73.3)
            uint32_t row = 2 * p + odd;
            __asm__ volatile("" : "+v"(row) : "v"(mag[0]));
            const float v[8] = {A[2 * p].x,     A[2 * p].y,     A[2 * p].z,     A[2 * p].w,
                                A[2 * p + 1].x, A[2 * p + 1].y, A[2 * p + 1].z, A[2 * p + 1].w};
            const bool rare = fast_mags(v, inv8, c.s0x, lk, tab.key[row], key0, key1, bits, mag, sgn);
            redo |= rare || !c.pre ? 1u << p : 0u;
            use(p, mag, sgn, nullptr);
        }
    }
    // the pairs that need it once more, from memory (a loop here instead of a
    // branch per pair keeps the tile's code straight and a third of the size)
    while (__builtin_expect(redo != 0u, 0)) {
        const int p = __builtin_ctz(redo);
        redo &= redo - 1u;
        f32x4 B[2];
        const int32_t r0 = 2 * p;
        load_quads<2, TAIL>(g + static_cast<int64_t>(r0) * ldg, ldg, rows - r0 < 2 ? 1 : 2, T, d, B);
        const float v[8] = {B[0].x, B[0].y, B[0].z, B[0].w, B[1].x, B[1].y, B[1].z, B[1].w};
        fast_mags(v, inv8, c.s0x, lk, tab.key[2 * p + odd], key0, key1, bits, mag, sgn);
        u16x2 ex[4];
        exact_mags(v, inv8, c.s0x, c.pre, c0, c1, worker0 + 2u * p + odd, key0, key1, bits, ex);
        use(p, ex, sgn, mag);
    }
}

template <int BITS>
__device__ __forceinline__ void lds_put(uint8_t* p, uint32_t v)
{
    if (BITS == 8)
        *reinterpret_cast<uint32_t*>(p) = v;
    else if (BITS == 4)
        *reinterpret_cast<uint16_t*>(p) = static_cast<uint16_t>(v);
    else
        *p = static_cast<uint8_t>(v);
}

// What a rows pass writes: the index (several scales), the rows' codes as
// BITS-bit fields (BITS = 0: not stored), and, unless sum is null, their
// sums and the reconstruction.
struct RowsOut {
    uint8_t* idx;
    uint8_t* codes;
    int64_t ldc;
    int32_t* sum;
    float* out;
};

constexpr int rows_stage_bytes(int rows, int bits)
{
    return rows * 32 * bits < 16 ? 16 : rows * 32 * bits;
}

// One tile: the index, every row's codes (collected in the wave's LDS rows
// `stage` and stored as 16-byte pieces), their sums in 16-bit lanes (|sum| <=
// 16 * 127, exact) and the reconstruction.
template <int ROWS, bool MULTI, int BITS, int POL, bool TAIL>
__device__ __forceinline__ void rows_tile(const f32x4 (&A)[ROWS], const float* __restrict__ g, int64_t ldg,
                                          int32_t rows, uint32_t worker0, int64_t T, int64_t d, const WaveScale& c,
                                          int32_t K, const RowTables& tab, uint32_t key0, uint32_t key1,
                                          const RowsOut& o, uint8_t* stage)
{
    constexpr int kRowBytes = 32 * BITS;  // one row's codes of a tile
    const int lane = threadIdx.x & 63;
    const int64_t a_off = T << 8;
    const int64_t left = TAIL ? d - a_off - 4 * lane : 4;
    uint32_t k[4] = {0u, 0u, 0u, 0u};
    if (MULTI) {
        quad_index<ROWS>(A, c, K, k);
        store_index<TAIL>(o.idx, T, d, k);
    }
    float inv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        inv[j] = MULTI ? tab.inv[k[j]] : lane_value(c.inv, 0);
    u16x2 h0 = {0, 0}, h1 = {0, 0};
    for_row_pairs<ROWS, TAIL>(
        A, g, ldg, rows, worker0, T, d, c, inv, tab, key0, key1,
        [&](int p, const u16x2 mag[4], const u16x2 sgn[4], const u16x2* fast) {
            if (BITS != 0) {
                uint32_t q[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    q[j] = __builtin_bit_cast(uint32_t, static_cast<u16x2>(mag[j] * sgn[j]));
                constexpr int B = BITS == 0 ? 8 : BITS;
                uint8_t* srow = stage + 2 * p * kRowBytes + lane * (B / 2);
                lds_put<B>(srow, pack_quad<B>(q[0], q[1]));
                lds_put<B>(srow + kRowBytes, pack_quad<B>(q[2], q[3]));
            }
            u16x2 m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                m[j] = fast ? static_cast<u16x2>(mag[j] - fast[j]) : mag[j];
            add_pair(m, sgn, 2 * p + 1 < rows, h0, h1);
        });
    if (BITS != 0) {
        // the wave's own LDS writes complete before the reads below
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!TAIL) {
            // 16-byte pieces, several rows' per store
            constexpr int kPieces = BITS == 0 ? 1 : kRowBytes / 16;
            constexpr int kAll = ROWS * kPieces;
#pragma unroll
            for (int p0 = 0; p0 < kAll; p0 += 64) {
                const int p = p0 + lane;
                const int r = p / kPieces;
                const int off = (p % kPieces) * 16;
                if (p < kAll && r < rows) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + r * kRowBytes + off);
                    u32x4* dst = reinterpret_cast<u32x4*>(o.codes + static_cast<int64_t>(r) * o.ldc + T * kRowBytes + off);
                    if (POL != 0)
                        __builtin_nontemporal_store(v, dst);
                    else
                        *dst = v;
                }
            }
        } else {
            // the row's bytes up to d (int8), or those of every 8-coordinate
            // group that starts below d (fields past d hold 0)
            const int64_t rest = d - a_off;
            const int64_t n = BITS == 8 ? rest : (rest + 7) / 8 * BITS;
            for (int32_t r = 0; r < rows; ++r)
                for (int64_t i = lane; i < n; i += 64)
                    o.codes[static_cast<int64_t>(r) * o.ldc + T * kRowBytes + i] = stage[r * kRowBytes + i];
        }
        if (o.sum == nullptr)
            return;
    }
    const i32x4 s = {static_cast<int16_t>(h0.x), static_cast<int16_t>(h0.y), static_cast<int16_t>(h1.x),
                     static_cast<int16_t>(h1.y)};
    const float deq0 = lane_value(c.deq, 0);
    f32x4 r;
    r.x = static_cast<float>(s.x) * (MULTI ? tab.deq[k[0]] : deq0);
    r.y = static_cast<float>(s.y) * (MULTI ? tab.deq[k[1]] : deq0);
    r.z = static_cast<float>(s.z) * (MULTI ? tab.deq[k[2]] : deq0);
    r.w = static_cast<float>(s.w) * (MULTI ? tab.deq[k[3]] : deq0);
    if (left >= 4) {
        if (POL == kStoreNontemporal) {
            __builtin_nontemporal_store(s, reinterpret_cast<i32x4*>(o.sum + a_off + 4 * lane));
            store_nt(o.out + a_off + 4 * lane, r);
        } else {
            store_through<POL == kStoreBoth>(o.sum + a_off, 16 * lane, s);
            if (POL == kStoreSumsThrough || (MULTI && POL == kStoreThrough))
                store_nt(o.out + a_off + 4 * lane, r);
            else
                store_through<POL == kStoreBoth>(o.out + a_off, 16 * lane, r);
        }
    } else {
        const int64_t i = a_off + 4 * lane;
        if (left > 0) { o.sum[i] = s.x; o.out[i] = r.x; }
        if (left > 1) { o.sum[i + 1] = s.y; o.out[i + 1] = r.y; }
        if (left > 2) { o.sum[i + 2] = s.z; o.out[i + 2] = r.z; }
    }
}

// Where a rows pass takes W from: *w, or (part not null) the norm's chunk
// partials [rows][nchunks], reduced by every wave for itself in k_finish's
// order; the first block then also stores it to *w.
struct WSource {
    float* w;
    const double* part;
    int32_t nchunks;
};

// Partials per row up to which a wave reduces them itself: two loads a lane.
constexpr int32_t kOwnChunks = 128;

// This lane's part of each row's sum (partials lane and lane + 64).
template <int ROWS>
__device__ __forceinline__ void load_partials(const WSource& src, int32_t rows, double (&s)[ROWS])
{
    const int lane = threadIdx.x & 63;
    double x[ROWS], y[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double* p = src.part + static_cast<int64_t>(r < rows ? r : 0) * src.nchunks;
        x[r] = lane < src.nchunks ? p[lane] : 0.0;
        y[r] = lane + 64 < src.nchunks ? p[lane + 64] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        s[r] = r < rows ? x[r] + y[r] : 0.0;
}

// Has the lane sums formed (and so their loads waited for) where it stands,
// before the rows' loads go out: left to the reduction, they would be waited
// for together with the rows (2^20 coordinates of 4 rows: the step 13.4 us,
// 12.6 this way).
template <int ROWS>
__device__ __forceinline__ void settle(double (&s)[ROWS])
{
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        __asm__ volatile("" : "+v"(s[r]));
}

// One step of the rows' butterfly at distance `off` over N registers: row
// pairs are sent to the two halves that have become equal, so that the next
// distance works on half the registers.
template <int N>
__device__ __forceinline__ void fold_rows(double* s, int off)
{
    const bool upper = (threadIdx.x & off) != 0;
    if (N == 1) {
        s[0] += __shfl_xor(s[0], off, 64);
    } else {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const double keep = upper ? s[2 * i + 1] : s[2 * i];
            const double send = upper ? s[2 * i] : s[2 * i + 1];
            s[i] = keep + __shfl_xor(send, off, 64);
        }
    }
}

// The largest sum of squares of the rows from their lane sums (NaN if a row's
// is): each row's butterfly over distances 32 .. 1 (k_finish's order), several
// rows at a time, then their largest.
template <int ROWS>
__device__ __forceinline__ double largest_row(const double (&in)[ROWS])
{
    constexpr int N0 = ROWS <= 2 ? 2 : ROWS <= 4 ? 4 : ROWS <= 8 ? 8 : 16;
    double s[N0];
#pragma unroll
    for (int r = 0; r < N0; ++r)
        s[r] = r < ROWS ? in[r < ROWS ? r : 0] : 0.0;
    fold_rows<N0>(s, 32);
    fold_rows<(N0 > 2 ? N0 / 2 : 1)>(s, 16);
    fold_rows<(N0 > 4 ? N0 / 4 : 1)>(s, 8);
    fold_rows<(N0 > 8 ? N0 / 8 : 1)>(s, 4);
    fold_rows<1>(s, 2);
    fold_rows<1>(s, 1);
    const bool any_nan = __ballot(s[0] != s[0]) != 0;
    double best = s[0] > 0.0 ? s[0] : 0.0;
#pragma unroll
    for (int off = 32; off >= 4; off >>= 1) {
        const double o = __shfl_xor(best, off, 64);
        best = o > best ? o : best;
    }
    return any_nan ? __builtin_nan("") : best;
}

// Block b takes tile tile0 + b; the tile past the whole ones holds the last
// coordinates.  There is no loop over tiles: with one, the compiler kept the
// rows' keys and other loop invariants in registers and held far more of them;
// a call with more tiles than the grid cap is several launches.
// NORM: W from memory, from the partials, or by a run-time branch.  With one
// scale and no codes stored the two are compiled apart, because the partials'
// reduction takes registers beside the rows (8 rows 96 without, 102 with; 4
// rows 80 and 86): 5 rows of 5.0 M coordinates 43.7 us with the branch, 42.7
// without.  So are up to 4 rows of stored codes (25.6 M coordinates, four
// scales: one row 46.3 us with the branch, 44.9 without, 3 rows 80.5 and
// 78.1).  The rest keep the branch: apart they were no faster, 16 rows of
// VGG-16 size 0.3% slower, with 4-bit codes 0.7%.
constexpr int kNormRead = 0, kNormOwn = 1, kNormEither = 2;
template <int ROWS, bool MULTI, int BITS, int POL, int NORM>
__device__ __forceinline__ void rows_block(const float* __restrict__ g, int64_t d, int32_t rows, int64_t ldg,
                                           int32_t worker0, const WSource& src, const ScaleSet& S, uint32_t key0,
                                           uint32_t key1, int64_t tile0, int32_t M, const RowsOut& o)
{
    __shared__ RowTables tab;
    __shared__ __align__(16) uint8_t stage[rows_stage_bytes(ROWS, BITS)];
    int64_t T = tile0 + blockIdx.x;
    if (BITS == 2) {
        // a row's codes of a tile are half a 128-byte line: adjacent tiles
        // to blocks 8 apart, which the same XCD runs, so that its L2 joins
        // the halves
        const uint32_t b = blockIdx.x;
        if ((b | 15u) < gridDim.x)
            T = tile0 + ((b & ~15u) | ((b & 7u) << 1) | ((b >> 3) & 1u));
    }
    const bool whole = T < d >> 8;
    const bool own = NORM == kNormOwn || (NORM == kNormEither && src.part != nullptr);
    // the partials go out before the rows, whose loads they would wait behind
    double part[ROWS];
    if (own)
        load_partials<ROWS>(src, rows, part);
    if (NORM == kNormOwn)
        settle<ROWS>(part);
    f32x4 A[ROWS];
    if (whole)
        load_quads<ROWS, false>(g, ldg, rows, T, d, A);
    if (threadIdx.x < ROWS)
        tab.key[threadIdx.x] = row_key(quad_c1(T), static_cast<uint32_t>(worker0) + threadIdx.x, key0);
    float W;
    if (own) {
        W = static_cast<float>(sqrt(largest_row<ROWS>(part)));
        if (T == 0 && threadIdx.x == 0)
            *src.w = W;
    } else {
        W = *src.w;
    }
    const WaveScale c = wave_scale<MULTI>(W, S, M);
    if (MULTI && threadIdx.x < kMaxScales) {
        tab.inv[threadIdx.x] = c.inv;
        tab.deq[threadIdx.x] = c.deq;
    }
    __syncthreads();
    if (whole) {
        rows_tile<ROWS, MULTI, BITS, POL, false>(A, g, ldg, rows, static_cast<uint32_t>(worker0), T, d, c, S.K, tab,
                                                key0, key1, o, stage);
    } else {
        load_quads<ROWS, true>(g, ldg, rows, T, d, A);
        rows_tile<ROWS, MULTI, BITS, POL, true>(A, g, ldg, rows, static_cast<uint32_t>(worker0), T, d, c, S.K, tab,
                                               key0, key1, o, stage);
    }
}

// With many rows fewer waves per SIMD than fit.  More than 12 rows: two (16
// rows of VGG-16 size ran in 1.66 ms with two waves and 1.68-1.70 with three;
// 4-bit codes stored: 1.80 and 1.87); one scale from 11 rows (12 rows, steps
// in a loop over three sets of buffers: 7.0 M coordinates 119.2 us with four
// waves, 117.2 with two; 11.2 M 186.4 and 181.8; 3.0 M 56.0 and 56.6).  7 to
// 12 rows: four (8 rows of 11.2 M: 128.4 us with five, 127.4 with four; of
// 25.6 M 157-170 with four or five and 170-195 with two).
#define UQ_ROWS_WAVES(ROWS, TWO) \
    __attribute__((amdgpu_waves_per_eu(1, (ROWS) >= (TWO) ? 2 : (ROWS) > 6 ? 4 : 8)))

// One scale, no codes stored.
template <int ROWS, int POL, bool OWN>
__global__ __launch_bounds__(64) UQ_ROWS_WAVES(ROWS, 11) void k_quant_sum_split(
    const float* __restrict__ g, int64_t d, int32_t rows, int64_t ldg, int32_t worker0, WSource src, ScaleSet S,
    uint32_t key0, uint32_t key1, int64_t tile0, int32_t M, RowsOut o)
{
    rows_block<ROWS, false, 0, POL, OWN ? kNormOwn : kNormRead>(g, d, rows, ldg, worker0, src, S, key0, key1, tile0, M, o);
}

// The same with a tile's rows split over the block's four waves: wave w codes rows w * RPW .. + RPW - 1 (and with OWN reduces their
// partials), the waves' sums meet in LDS, wave 0 stores the tile's sums and
// wave 1 its outputs.  One wave holding every row leaves a SIMD two waves at
// 11 rows and more, and few tiles fill those unevenly: 16 rows of 262,144
// coordinates 13.9 us with one wave, 12.0 with four; 524,288 21.3 and 19.9;
// 2^20 34.4 and 33.6; 12 rows 2^20 27.1 and 25.9; from 2^21 on the two are
// equal, and with 9 or 10 rows one wave is faster (0.8 M 17.4 and 19.5).
// 8 rows, two a wave: 5.0 M coordinates 62.7 and 61.8 us, 9.0 M 104.0 and
// 101.7, 11.2 M 128.3 and 125.5 (3.1 M 43.0 and 43.5; fewer rows leave a wave
// a single one: 7 rows' pass alone, in cache, 62.0 and 64.0, 5 rows' step 85.0
// and 91.0).
template <int RPW, bool OWN>
__global__ __launch_bounds__(256) void k_quant_sum_waves(
    const float* __restrict__ g, int64_t d, int32_t rows, int64_t ldg, int32_t worker0, WSource src, ScaleSet S,
    uint32_t key0, uint32_t key1, int64_t tile0, int32_t M, RowsOut o)
{
    __shared__ RowTables tab_s[4];
    __shared__ uint2 part_s[4][64];
    __shared__ double best_s[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    const int64_t T = tile0 + blockIdx.x;
    const bool whole = T < d >> 8;
    // the wave's rows r0 .. r0 + n - 1 (none: it reads the last row and adds nothing)
    const int32_t r0 = wave * RPW < rows ? wave * RPW : rows - 1;
    const int32_t n = wave * RPW < rows ? (rows - r0 < RPW ? rows - r0 : RPW) : 0;
    const int32_t n_read = n > 0 ? n : 1;
    const float* mine = g + static_cast<int64_t>(r0) * ldg;
    const uint32_t first = static_cast<uint32_t>(worker0) + static_cast<uint32_t>(r0);
    double part[RPW];
    if (OWN) {
        load_partials<RPW>(WSource{nullptr, src.part + static_cast<int64_t>(r0) * src.nchunks, src.nchunks}, n_read,
                           part);
        settle<RPW>(part);
    }
    f32x4 A[RPW];
    if (whole)
        load_quads<RPW, false>(mine, ldg, n_read, T, d, A);
    else
        load_quads<RPW, true>(mine, ldg, n_read, T, d, A);
    RowTables& tab = tab_s[wave];
    if (lane < RPW)
        tab.key[lane] = row_key(quad_c1(T), first + static_cast<uint32_t>(lane), key0);
    float W;
    if (OWN) {
        const double best = largest_row<RPW>(part);
        if (lane == 0)
            best_s[wave] = best;
        __syncthreads();
        bool any_nan = false;
        double most = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            any_nan = any_nan || best_s[w] != best_s[w];
            most = best_s[w] > most ? best_s[w] : most;
        }
        W = any_nan ? __builtin_nanf("") : static_cast<float>(sqrt(most));
        if (T == 0 && threadIdx.x == 0)
            *src.w = W;
    } else {
        W = *src.w;
    }
    const WaveScale c = wave_scale<false>(W, S, M);
    const float inv0 = lane_value(c.inv, 0);
    const float inv[4] = {inv0, inv0, inv0, inv0};
    // the wave's own keys are in LDS before it reads them
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    u16x2 h0 = {0, 0}, h1 = {0, 0};
    const auto add = [&](int p, const u16x2 mag[4], const u16x2 sgn[4], const u16x2* fast) {
        u16x2 m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            m[j] = fast ? static_cast<u16x2>(mag[j] - fast[j]) : mag[j];
        add_pair(m, sgn, 2 * p + 1 < n, h0, h1);
    };
    if (whole)
        for_row_pairs<RPW, false>(A, mine, ldg, n, first, T, d, c, inv, tab, key0, key1, add);
    else
        for_row_pairs<RPW, true>(A, mine, ldg, n, first, T, d, c, inv, tab, key0, key1, add);
    part_s[wave][lane] = make_uint2(__builtin_bit_cast(uint32_t, h0), __builtin_bit_cast(uint32_t, h1));
    __syncthreads();
    if (wave > 1)
        return;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w != wave) {
            const uint2 q = part_s[w][lane];
            h0 += __builtin_bit_cast(u16x2, q.x);
            h1 += __builtin_bit_cast(u16x2, q.y);
        }
    }
    const i32x4 s = {static_cast<int16_t>(h0.x), static_cast<int16_t>(h0.y), static_cast<int16_t>(h1.x),
                     static_cast<int16_t>(h1.y)};
    const float deq0 = lane_value(c.deq, 0);
    const f32x4 r = {static_cast<float>(s.x) * deq0, static_cast<float>(s.y) * deq0, static_cast<float>(s.z) * deq0,
                     static_cast<float>(s.w) * deq0};
    const int64_t i = (T << 8) + 4 * lane;
    const int64_t left = d - i;
    if (left >= 4) {
        if (wave == 0)
            store_through<false>(o.sum + (T << 8), 16 * lane, s);
        else
            store_through<false>(o.out + (T << 8), 16 * lane, r);
    } else {
        for (int j = 0; j < 3; ++j) {
            if (j < left) {
                if (wave == 0)
                    o.sum[i + j] = s[j];
                else
                    o.out[i + j] = r[j];
            }
        }
    }
}

// Several scales, no codes stored; the shared index formed and stored: all M
// rows, as workers 0 .. M - 1.
template <int ROWS, int POL>
__global__ __launch_bounds__(64) UQ_ROWS_WAVES(ROWS, 13) void k_index_quant_sum(
    const float* __restrict__ g, int64_t d, int32_t M, int64_t ldg, WSource src, ScaleSet S, uint32_t key0,
    uint32_t key1, int64_t tile0, RowsOut o)
{
    rows_block<ROWS, true, 0, POL, kNormEither>(g, d, M, ldg, 0, src, S, key0, key1, tile0, M, o);
}

// The codes stored as BITS-bit fields, and (o.sum not null) summed and
// reconstructed in the same pass, so that they are not read again.  OWN (up to
// 4 rows only): W from the partials; beyond, either way (see NORM).
template <int ROWS, bool MULTI, int BITS, bool NT, bool OWN>
__global__ __launch_bounds__(64) UQ_ROWS_WAVES(ROWS, 13) void k_index_quantise(
    const float* __restrict__ g, int64_t d, int32_t M, int64_t ldg, WSource src, ScaleSet S, uint32_t key0,
    uint32_t key1, int64_t tile0, RowsOut o)
{
    constexpr int kNorm = ROWS > 4 || OWN ? kNormEither : kNormRead;
    rows_block<ROWS, MULTI, BITS, NT ? kStoreBoth : kStoreThrough, kNorm>(g, d, M, ldg, 0, src, S, key0, key1, tile0,
                                                                          M, o);
}

// ---------------------------------------------------------------------------
// A whole step in one block, for d <= small_step(M) coordinates of at most 16
// rows: the rows' sums of squares in k_sumsq's order (one chunk a row: 256
// threads), W by k_finish's rule, then one wave per 256-coordinate tile as
// above.  At such sizes a step is launches and their latency.
// 1000 coordinates of 8 rows, codes stored: 24.0 us as four kernels, 11.9 as one.
// ---------------------------------------------------------------------------
constexpr int kSmallThreads = 512;
// The one block codes its rows in turn, so more rows leave it fewer
// coordinates before norm and rows pass over many blocks (12.3 us, 8 to 16
// rows) are faster: 8 rows of 4096 9.9 us (four scales 11.6); 16 rows of 2048
// 12.1 (12.9), of 3072 14.6 (15.9), of 4096 18.6 (20.2).
constexpr int64_t kSmallStep = 4096;
constexpr int64_t small_step(int32_t rows)
{
    return rows <= 8 ? kSmallStep : kSmallStep / 2;
}

template <int ROWS, bool MULTI, int BITS>
__global__ __launch_bounds__(kSmallThreads) void k_step_small(const float* __restrict__ g, int64_t d, int32_t M,
                                                              int64_t ldg, float* __restrict__ w, ScaleSet S,
                                                              uint32_t key0, uint32_t key1, RowsOut o)
{
    __shared__ double wave_part[ROWS][4];
    __shared__ RowTables tab;
    __shared__ __align__(16) uint8_t stage_s[kSmallThreads / 64][rows_stage_bytes(ROWS, BITS)];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x >> 6));
    // two rows at a time, 256 threads each
    const int32_t nvec = static_cast<int32_t>(d >> 2);
    const int t = threadIdx.x & 255;
    double sq[ROWS / 2];
#pragma unroll
    for (int i = 0; i < ROWS / 2; ++i) {
        const int m = 2 * i + static_cast<int>(threadIdx.x >> 8);
        const float* row = g + static_cast<int64_t>(m < M ? m : M - 1) * ldg;
        double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
#pragma unroll
        for (int u = 0; u < small_step(ROWS) / 1024; ++u) {
            const int32_t j = t + 256 * u;
            if (j < nvec) {
                const f32x4 a = *reinterpret_cast<const f32x4*>(row + 4 * j);
                acc0 = fma((double)a.x, (double)a.x, acc0); acc1 = fma((double)a.y, (double)a.y, acc1);
                acc2 = fma((double)a.z, (double)a.z, acc2); acc3 = fma((double)a.w, (double)a.w, acc3);
            }
        }
        const int32_t tail = 4 * nvec + t;
        if (tail < d) {
            const double x = row[tail];
            acc0 = fma(x, x, acc0);
        }
        sq[i] = (acc0 + acc1) + (acc2 + acc3);
    }
#pragma unroll
    for (int i = 0; i < ROWS / 2; ++i) {
        const double s = wave_sum(sq[i]);
        if (lane == 0)
            wave_part[2 * i + (wave >> 2)][wave & 3] = s;
    }
    __syncthreads();
    double best = 0.0;
    bool any_nan = false;
    for (int32_t m = 0; m < M; ++m) {
        const double r = (wave_part[m][0] + wave_part[m][1]) + (wave_part[m][2] + wave_part[m][3]);
        any_nan = any_nan || (r != r);
        best = r > best ? r : best;
    }
    const float W = any_nan ? __builtin_nanf("") : static_cast<float>(sqrt(best));
    if (threadIdx.x == 0)
        *w = W;
    const WaveScale c = wave_scale<MULTI>(W, S, M);
    if (threadIdx.x < ROWS)
        tab.key[threadIdx.x] = row_key(0u, threadIdx.x, key0);
    if (MULTI && threadIdx.x < kMaxScales) {
        tab.inv[threadIdx.x] = c.inv;
        tab.deq[threadIdx.x] = c.deq;
    }
    __syncthreads();
    for (int32_t T = wave; T < (d + 255) >> 8; T += kSmallThreads / 64) {
        f32x4 A[ROWS];
        if (T < d >> 8) {
            load_quads<ROWS, false>(g, ldg, M, T, d, A);
            rows_tile<ROWS, MULTI, BITS, kStoreThrough, false>(A, g, ldg, M, 0u, T, d, c, S.K, tab, key0, key1, o,
                                                       stage_s[wave]);
        } else {
            load_quads<ROWS, true>(g, ldg, M, T, d, A);
            rows_tile<ROWS, MULTI, BITS, kStoreThrough, true>(A, g, ldg, M, 0u, T, d, c, S.K, tab, key0, key1, o,
                                                      stage_s[wave]);
        }
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers (called by the ABI layer after validation).
// ---------------------------------------------------------------------------
// A launch that stores codes stores them nontemporally when it writes more
// than this many bytes: measured 3% faster steps at VGG-16 size (2.2 GB of
// codes), 1.8-2.5% slower at ResNet-18 and ResNet-50 sizes (89 and 204 MB),
// where the sum then finds the codes in the 256 MB Infinity Cache.
constexpr int64_t kCodesNontemporalBytes = int64_t(512) << 20;

// Enough blocks for every unit to get its own thread / wave / tile (the
// streaming kernels run fastest as one pass with no grid-stride reuse).  The
// dispatch packet counts work-items in 32 bits, so the grid is capped at 2^22
// blocks.  What one grid does not cover, the one-wave kernels (one block per
// tile) take in further launches, past 2^30 coordinates at the earliest, and
// the others in grid-stride loops.  Tests lower the cap to reach both at small
// sizes.
constexpr int64_t kMaxBlocks = int64_t(1) << 22;
static std::atomic<int64_t> g_one_shot_cap{kMaxBlocks};

bool set_one_shot_cap(int64_t blocks)
{
    if (blocks == 0)
        blocks = kMaxBlocks;
    if (blocks < kMinOneShotCap || blocks > kMaxBlocks)
        return false;
    g_one_shot_cap.store(blocks, std::memory_order_relaxed);
    return true;
}

static int64_t one_shot_cap()
{
    return g_one_shot_cap.load(std::memory_order_relaxed);
}

// One launch's share of `units` one-unit blocks from `first` on, at most `cap`.
static unsigned blocks_from(int64_t units, int64_t first, int64_t cap)
{
    return static_cast<unsigned>(units - first < cap ? units - first : cap);
}

static unsigned one_shot(int64_t units, int64_t per_block)
{
    const int64_t cap = one_shot_cap();
    int64_t blocks = (units + per_block - 1) / per_block;
    blocks = blocks < 1 ? 1 : (blocks > cap ? cap : blocks);
    return static_cast<unsigned>(blocks);
}

// The fused pass stores the row maxima's keys nontemporally when they exceed
// this many bytes: measured 5% faster (the shared scale) at VGG-16 size
// (277 MB of keys), 3% slower at ResNet-50 size (51 MB), where the index pass
// reads them back from the 256 MB Infinity Cache.
constexpr int64_t kMaximaNontemporalBytes = int64_t(128) << 20;
// The index pass stores the index (one byte per coordinate) nontemporally
// beyond this many bytes, where the passes that read it back find it in HBM.
constexpr int64_t kIndexNontemporalBytes = int64_t(256) << 20;

// One scale's rows pass stores its outputs nontemporally beyond this many
// bytes of them (between 11.2 M and 12.5 M coordinates) and its sums beyond
// kSumsThroughBytes (between 20.0 M and 25.6 M; see kStoreThrough).
constexpr int64_t kOutNontemporalBytes = int64_t(46) << 20;
constexpr int64_t kSumsThroughBytes = int64_t(88) << 20;
// The one-row quantise-and-sum leaves its sums in the XCDs' L2s (4 MB each)
// up to this many bytes of them, where the next worker's call finds them: 8
// streamed workers, one scale, 4.2 M coordinates 99.9 us written through, 89.3
// plain; 6.3 M 140.4 and 123.9; 8.4 M 173.1 and 174.9 (four scales 213 and
// 221).  Its outputs leave nontemporally beyond kOutNontemporalBytes: one
// worker of 16.0 M coordinates 48.4 us through, 41.7.
constexpr int64_t kSumsInL2Bytes = int64_t(28) << 20;
// Write-through stores also carry the nontemporal hint when the sums exceed
// this many bytes, the Infinity Cache's size (work-free passes): the sums and
// outputs of 16 rows at VGG-16 size, with the index, 1.64 against 1.72 ms;
// at ResNet-50 size (102 MB) 167 us with the hint, 157 without.
constexpr int64_t kThroughNontemporalBytes = int64_t(256) << 20;

// The norm: chunk partials, and W from them unless w is null.
static hipError_t launch_norm(const float* g, int64_t d, int32_t M, int64_t ldg, const NormPlan& plan, float* w,
                              double* part, hipStream_t stream)
{
    if (plan.nchunks > 0) {
        // rows beyond the grid cap / nchunks are taken in turn by the same blocks
        int64_t gy = one_shot_cap() / plan.nchunks;
        gy = gy < 1 ? 1 : (gy > M ? M : gy);
        dim3 grid(static_cast<unsigned>(plan.nchunks), static_cast<unsigned>(gy));
        hipLaunchKernelGGL(k_sumsq, grid, dim3(kBlock), 0, stream, g, d, M, ldg, plan.chunk, plan.nchunks, part);
    }
    if (w != nullptr)
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(kFinishThreads), 0, stream, part, plan.nchunks, M, w);
    return hipGetLastError();
}

hipError_t launch_shared_scale(const float* g, int64_t d, int32_t M, int64_t ldg, const ScaleSet& S,
                               float* w, uint8_t* idx, void* ws, hipStream_t stream, int32_t idx_bits)
{
    const bool nib = idx_bits == 4;
    if (use_fused(d, M, S.K)) {
        const FusedPlan plan = fused_plan(d);
        const FusedLayout L = fused_layout(d, M);
        double* part = static_cast<double*>(ws);
        double* sub = reinterpret_cast<double*>(static_cast<char*>(ws) + L.sub_off);
        double* rows = reinterpret_cast<double*>(static_cast<char*>(ws) + L.rows_off);
        IndexTables* tabs = reinterpret_cast<IndexTables*>(static_cast<char*>(ws) + L.tab_off);
        uint16_t* keys = fused_keys(ws, L);
        const dim3 grid(one_shot(plan.ntiles + 1, 1));
        // keys beyond half the 256 MB Infinity Cache are stored
        // nontemporally (the index pass would not find them there)
        const bool nt = 2 * d > kMaximaNontemporalBytes;
        const bool one = static_cast<int64_t>(grid.x) >= plan.ntiles + 1;
#define UQ_LAUNCH_NORM_MAX_(R, NT)                                                                                \
    do {                                                                                                          \
        if (one)                                                                                                  \
            hipLaunchKernelGGL((k_norm_max<R, NT, true>), grid, dim3(kBlock), 0, stream, g, d, M, ldg,            \
                               plan.ntiles, part, keys);                                                          \
        else                                                                                                      \
            hipLaunchKernelGGL((k_norm_max<R, NT, false>), grid, dim3(kBlock), 0, stream, g, d, M, ldg,           \
                               plan.ntiles, part, keys);                                                          \
    } while (0)
#define UQ_LAUNCH_NORM_MAX(R)              \
    do {                                   \
        if (nt)                            \
            UQ_LAUNCH_NORM_MAX_(R, true);  \
        else                               \
            UQ_LAUNCH_NORM_MAX_(R, false); \
    } while (0)
        if (M <= 4)
            UQ_LAUNCH_NORM_MAX(4);
        else if (M <= 8)
            UQ_LAUNCH_NORM_MAX(8);
        else
            UQ_LAUNCH_NORM_MAX(kFuseRows);
#undef UQ_LAUNCH_NORM_MAX
#undef UQ_LAUNCH_NORM_MAX_
        // the rows' sums: kRowsumSpan tile partials at a time, then those sums
        hipLaunchKernelGGL(k_rowsum, dim3(static_cast<unsigned>(plan.nsub), static_cast<unsigned>(M)), dim3(kBlock),
                           0, stream, part, plan.ntiles + 1, kRowsumSpan, sub);
        // then S_m, W and the index pass's constants in one block
        hipLaunchKernelGGL(k_index_prep, dim3(1), dim3(kBlock), 0, stream, sub, plan.nsub, M, rows, w, S, tabs);
        const unsigned gx = one_shot((d + 7) / 8, kIndexTile);
#define UQ_LAUNCH_INDEX_MAX(NT, NIB)                                                                            \
    hipLaunchKernelGGL((k_index_max<NT, NIB>), dim3(gx), dim3(kBlock), 0, stream, keys, g, ldg, d, M, tabs, S.K, idx)
        // the index is stored nontemporally beyond kIndexNontemporalBytes
        if ((nib ? (d + 1) / 2 : d) > kIndexNontemporalBytes) {
            if (nib) UQ_LAUNCH_INDEX_MAX(true, true); else UQ_LAUNCH_INDEX_MAX(true, false);
        } else {
            if (nib) UQ_LAUNCH_INDEX_MAX(false, true); else UQ_LAUNCH_INDEX_MAX(false, false);
        }
#undef UQ_LAUNCH_INDEX_MAX
        return hipGetLastError();
    }
    double* part = static_cast<double*>(ws);
    const hipError_t e = launch_norm(g, d, M, ldg, norm_plan(d), w, part, stream);
    if (e != hipSuccess)
        return e;
    if (S.K > 1 && d > 0) {
        const unsigned gx = one_shot((d + 3) / 4, kBlock);
        if (nib)
            hipLaunchKernelGGL(k_index<true>, dim3(gx), dim3(kBlock), 0, stream, g, d, M, ldg, w, S, idx);
        else
            hipLaunchKernelGGL(k_index<false>, dim3(gx), dim3(kBlock), 0, stream, g, d, M, ldg, w, S, idx);
    }
    return hipGetLastError();
}

hipError_t launch_quantise(const float* g, int64_t d, int32_t rows, int64_t ldg, int32_t worker0,
                           const float* w, const ScaleSet& S, const uint8_t* idx, uint64_t seed,
                           void* codes, int64_t ldc, int32_t bits, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    const uint32_t key0 = static_cast<uint32_t>(seed);
    const uint32_t key1 = static_cast<uint32_t>(seed >> 32);
    // one block per 512-coordinate tile and row (the last tile partial), rows
    // x tiles within the grid cap
    const int64_t ntiles = (d + 511) >> 9;
    const int64_t share = one_shot_cap() / rows;
    const int64_t per_row = share < 1 ? 1 : share;
    uint8_t* out = reinterpret_cast<uint8_t*>(codes);
    // (from 256 MB on, 16 rows of 25.6 M coordinates, 409 MB of codes, then
    // their sum, took 667 us; from 512 MB 641)
    const bool nt = static_cast<int64_t>(rows) * ((d * bits + 7) / 8) > kCodesNontemporalBytes;
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += per_row) {
        const dim3 grid(blocks_from(ntiles, tile0, per_row), static_cast<unsigned>(rows));
#define UQ_LAUNCH_QUANTISE(MULTI, BITS)                                                                            \
    do {                                                                                                           \
        if (nt)                                                                                                    \
            hipLaunchKernelGGL((k_quantise<MULTI, BITS, true>), grid, dim3(64), 0, stream, g, d, ldg, worker0, w,  \
                               S, idx, key0, key1, tile0, out, ldc);                                               \
        else                                                                                                       \
            hipLaunchKernelGGL((k_quantise<MULTI, BITS, false>), grid, dim3(64), 0, stream, g, d, ldg, worker0, w, \
                               S, idx, key0, key1, tile0, out, ldc);                                               \
    } while (0)
        const bool multi = S.K > 1;
        if (bits == 8) {
            if (multi) UQ_LAUNCH_QUANTISE(true, 8); else UQ_LAUNCH_QUANTISE(false, 8);
        } else if (bits == 4) {
            if (multi) UQ_LAUNCH_QUANTISE(true, 4); else UQ_LAUNCH_QUANTISE(false, 4);
        } else {
            if (multi) UQ_LAUNCH_QUANTISE(true, 2); else UQ_LAUNCH_QUANTISE(false, 2);
        }
    }
#undef UQ_LAUNCH_QUANTISE
    return hipGetLastError();
}

// The rows pass's stores by the bytes of its sums (see kStoreThrough), with
// several scales and with one.
static int rows_policy(int64_t d)
{
    return 4 * d > kThroughNontemporalBytes ? kStoreBoth : 4 * d > kSumNontemporalBytes ? kStoreNontemporal
                                                                                       : kStoreThrough;
}

static int one_scale_policy(int64_t d)
{
    return 4 * d > kThroughNontemporalBytes ? kStoreBoth
           : 4 * d > kSumsThroughBytes      ? kStoreNontemporal
           : 4 * d > kOutNontemporalBytes   ? kStoreSumsThrough
                                            : kStoreThrough;
}

// One scale, at most kFuseRows rows set and reconstructed in one call:
// one block per 256-coordinate tile (the last one partial), one instance per
// row pair count.
#define UQ_ROW_PAIRS_1_TO_8(LAUNCH, ...) \
    LAUNCH(1, __VA_ARGS__);              \
    LAUNCH(2, __VA_ARGS__);              \
    LAUNCH(3, __VA_ARGS__);              \
    LAUNCH(4, __VA_ARGS__);              \
    LAUNCH(5, __VA_ARGS__);              \
    LAUNCH(6, __VA_ARGS__);              \
    LAUNCH(7, __VA_ARGS__);              \
    LAUNCH(8, __VA_ARGS__)

// Tiles up to which 11 to 16 rows of one scale are split over four waves, and
// beyond which 8 are (up to kOutNontemporalBytes of outputs).
constexpr int64_t kWavesTiles = int64_t(1) << 13;
constexpr int64_t kPairTiles = int64_t(1) << 14;

static hipError_t launch_quant_sum_split(const float* g, int64_t d, int32_t rows, int64_t ldg, int32_t worker0,
                                         const WSource& src, const ScaleSet& S, uint32_t key0, uint32_t key1,
                                         int32_t M, const RowsOut& o, hipStream_t stream)
{
    const int64_t ntiles = (d + 255) >> 8;
    const bool few = rows > 10 && ntiles <= kWavesTiles;
    if (few || (rows == 8 && ntiles > kPairTiles && 4 * d <= kOutNontemporalBytes)) {
        const int64_t cap = one_shot_cap();
        for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
            const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_WAVES(RPW, OWN)                                                                                   \
    hipLaunchKernelGGL((k_quant_sum_waves<RPW, OWN>), grid, dim3(256), 0, stream, g, d, rows, ldg, worker0, src, S, \
                       key0, key1, tile0, M, o)
            // (the norm has too many partials for OWN where 8 rows come here)
            if (!few) UQ_LAUNCH_WAVES(2, false);
            else if (src.part != nullptr) UQ_LAUNCH_WAVES(4, true);
            else UQ_LAUNCH_WAVES(4, false);
#undef UQ_LAUNCH_WAVES
        }
        return hipGetLastError();
    }
    const int policy = one_scale_policy(d);
    const int64_t cap = one_shot_cap();
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_SPLIT(PAIRS, POL, OWN)                                                                           \
    case PAIRS:                                                                                                    \
        hipLaunchKernelGGL((k_quant_sum_split<2 * PAIRS, POL, OWN>), grid, dim3(64), 0, stream, g, d, rows, ldg,         \
                           worker0, src, S, key0, key1, tile0, M, o);                                              \
        break
        if (src.part != nullptr) {
            switch ((rows + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_SPLIT, kStoreThrough, true); }
        } else if (policy == kStoreThrough) {
            switch ((rows + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_SPLIT, kStoreThrough, false); }
        } else if (policy == kStoreSumsThrough) {
            switch ((rows + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_SPLIT, kStoreSumsThrough, false); }
        } else if (policy == kStoreNontemporal) {
            switch ((rows + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_SPLIT, kStoreNontemporal, false); }
        } else {
            switch ((rows + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_SPLIT, kStoreBoth, false); }
        }
#undef UQ_LAUNCH_SPLIT
    }
    return hipGetLastError();
}

hipError_t launch_quant_sum(const float* g, int64_t d, int32_t rows, int64_t ldg, int32_t worker0, const float* w,
                            const ScaleSet& S, const uint8_t* idx, uint64_t seed, int32_t accumulate, int32_t* sum,
                            int32_t M, float* out, hipStream_t stream, int32_t idx_bits)
{
    const bool nib = idx_bits == 4;
    if (d == 0)
        return hipSuccess;
    const uint32_t key0 = static_cast<uint32_t>(seed);
    const uint32_t key1 = static_cast<uint32_t>(seed >> 32);
    const bool nt = 4 * d > kThroughNontemporalBytes;
    const bool multi = S.K > 1;
    const bool acc = accumulate != 0;
    const bool deq = out != nullptr;
    const int32_t stores = 4 * d <= kSumsInL2Bytes ? kStorePlain : 4 * d > kOutNontemporalBytes ? kStoreSumsThrough
                                                                                               : kStoreThrough;
    if (!multi && !acc && deq && rows > 4 && rows <= kFuseRows)
        return launch_quant_sum_split(g, d, rows, ldg, worker0, WSource{const_cast<float*>(w), nullptr, 0}, S, key0,
                                      key1, M, RowsOut{nullptr, nullptr, 0, sum, out}, stream);
    // one block per 512-coordinate tile, the last one partial
    const int64_t ntiles = (d + 511) >> 9;
    const int64_t cap = one_shot_cap();
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_QSUM_(MULTI, ACC, DEQ, NT, NIB)                                                                   \
    do {                                                                                                           \
        if (rows == 1)                                                                                             \
            hipLaunchKernelGGL((k_quant_sum<MULTI, ACC, DEQ, NT, true, NIB>), grid, dim3(64), 0, stream, g, d,      \
                               rows, ldg, worker0, w, S, idx, key0, key1, tile0, sum, M, out, stores);                     \
        else                                                                                                       \
            hipLaunchKernelGGL((k_quant_sum<MULTI, ACC, DEQ, NT, false, NIB>), grid, dim3(64), 0, stream, g, d,     \
                               rows, ldg, worker0, w, S, idx, key0, key1, tile0, sum, M, out, stores);                     \
    } while (0)
    // the 4-bit index layout only matters with several scales (NIB = MULTI
    // there, so one scale compiles no second instance)
#define UQ_LAUNCH_QSUM(MULTI, ACC, DEQ, NT)                  \
    do {                                                     \
        if (nib)                                             \
            UQ_LAUNCH_QSUM_(MULTI, ACC, DEQ, NT, MULTI);     \
        else                                                 \
            UQ_LAUNCH_QSUM_(MULTI, ACC, DEQ, NT, false);     \
    } while (0)
#define UQ_LAUNCH_QSUM_NT(MULTI, ACC, DEQ)  \
    do {                                    \
        if (nt)                             \
            UQ_LAUNCH_QSUM(MULTI, ACC, DEQ, true);  \
        else                                \
            UQ_LAUNCH_QSUM(MULTI, ACC, DEQ, false); \
    } while (0)
#define UQ_LAUNCH_QSUM_DEQ(MULTI, ACC)           \
    do {                                         \
        if (deq)                                 \
            UQ_LAUNCH_QSUM_NT(MULTI, ACC, true); \
        else                                     \
            UQ_LAUNCH_QSUM_NT(MULTI, ACC, false);\
    } while (0)
        if (multi) {
            if (acc) UQ_LAUNCH_QSUM_DEQ(true, true); else UQ_LAUNCH_QSUM_DEQ(true, false);
        } else {
            if (acc) UQ_LAUNCH_QSUM_DEQ(false, true); else UQ_LAUNCH_QSUM_DEQ(false, false);
        }
    }
#undef UQ_LAUNCH_QSUM_DEQ
#undef UQ_LAUNCH_QSUM_NT
#undef UQ_LAUNCH_QSUM
#undef UQ_LAUNCH_QSUM_
    return hipGetLastError();
}

// Several scales, no codes stored: one block per 256-coordinate tile (the
// last one partial), one instance per row pair count.
static hipError_t launch_index_quant_sum_from(const float* g, int64_t d, int32_t M, int64_t ldg, const WSource& src,
                                              const ScaleSet& S, uint32_t key0, uint32_t key1, const RowsOut& o,
                                              hipStream_t stream)
{
    const int64_t ntiles = (d + 255) >> 8;
    const int policy = rows_policy(d);
    const int64_t cap = one_shot_cap();
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_IQS(PAIRS, POL)                                                                                  \
    case PAIRS:                                                                                                    \
        hipLaunchKernelGGL((k_index_quant_sum<2 * PAIRS, POL>), grid, dim3(64), 0, stream, g, d, M, ldg, src, S,    \
                           key0, key1, tile0, o);                                                                  \
        break
        if (policy == kStoreThrough) {
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQS, kStoreThrough); }
        } else if (policy == kStoreNontemporal) {
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQS, kStoreNontemporal); }
        } else {
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQS, kStoreBoth); }
        }
#undef UQ_LAUNCH_IQS
    }
    return hipGetLastError();
}

hipError_t launch_index_quant_sum(const float* g, int64_t d, int32_t M, int64_t ldg, const float* w,
                                  const ScaleSet& S, uint64_t seed, uint8_t* idx, int32_t* sum, float* out,
                                  hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    return launch_index_quant_sum_from(g, d, M, ldg, WSource{const_cast<float*>(w), nullptr, 0}, S,
                                       static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32),
                                       RowsOut{idx, nullptr, 0, sum, out}, stream);
}

// The codes stored as `bits`-bit fields (one scale or several), and summed
// and reconstructed too unless o.sum is null.
static hipError_t launch_stored_from(const float* g, int64_t d, int32_t M, int64_t ldg, const WSource& src,
                                     const ScaleSet& S, uint32_t key0, uint32_t key1, int32_t bits, const RowsOut& o,
                                     hipStream_t stream)
{
    const bool nt = static_cast<int64_t>(M) * ((d * bits + 7) / 8) > kCodesNontemporalBytes;
    const bool multi = S.K > 1 || o.idx != nullptr;
    const int64_t ntiles = (d + 255) >> 8;
    const int64_t cap = one_shot_cap();
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_IQ__(PAIRS, MULTI, BITS, NT, OWN)                                                                \
    hipLaunchKernelGGL((k_index_quantise<2 * PAIRS, MULTI, BITS, NT, OWN && (PAIRS <= 2)>), grid, dim3(64), 0,     \
                       stream, g, d, M, ldg, src, S, key0, key1, tile0, o)
#define UQ_LAUNCH_IQ_(PAIRS, BITS, NT, OWN)                \
    do {                                                   \
        if (multi)                                         \
            UQ_LAUNCH_IQ__(PAIRS, true, BITS, NT, OWN);    \
        else                                               \
            UQ_LAUNCH_IQ__(PAIRS, false, BITS, NT, OWN);   \
    } while (0)
#define UQ_LAUNCH_IQ(PAIRS, NT, OWN)              \
    case PAIRS:                                   \
        if (bits == 8)                            \
            UQ_LAUNCH_IQ_(PAIRS, 8, NT, OWN);     \
        else if (bits == 4)                       \
            UQ_LAUNCH_IQ_(PAIRS, 4, NT, OWN);     \
        else                                      \
            UQ_LAUNCH_IQ_(PAIRS, 2, NT, OWN);     \
        break
        if (src.part != nullptr) {
            // (at most 1024 partials: never codes of 512 MB)
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQ, false, true); }
        } else if (nt) {
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQ, true, false); }
        } else {
            switch ((M + 1) / 2) { UQ_ROW_PAIRS_1_TO_8(UQ_LAUNCH_IQ, false, false); }
        }
#undef UQ_LAUNCH_IQ
#undef UQ_LAUNCH_IQ_
#undef UQ_LAUNCH_IQ__
    }
    return hipGetLastError();
}

hipError_t launch_index_quantise(const float* g, int64_t d, int32_t M, int64_t ldg, const float* w,
                                 const ScaleSet& S, uint64_t seed, int32_t bits, uint8_t* idx, uint8_t* codes,
                                 int64_t ldc, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    return launch_stored_from(g, d, M, ldg, WSource{const_cast<float*>(w), nullptr, 0}, S, static_cast<uint32_t>(seed),
                              static_cast<uint32_t>(seed >> 32), bits, RowsOut{idx, codes, ldc, nullptr, nullptr},
                              stream);
}

// Partials (all rows') up to which every wave of the rows pass forms W from
// them itself instead of reading what k_finish formed, which takes a launch
// and a wait: with the partials and with k_finish, 4 rows of 128 each 12.3
// and 14.7 us, 8 rows of 64 13.1 and 15.0, of 128 (1024 in all) 19.8 and
// 20.5, 16 rows of 64 21.3 and 22.4.  The gain shrinks towards both limits;
// beyond them nothing was measured (more than 128 a row would take more than
// two loads a lane).
constexpr int64_t kOwnNormPartials = 1024;

static hipError_t launch_step_small(const float* g, int64_t d, int32_t M, int64_t ldg, float* w, const ScaleSet& S,
                                    uint32_t key0, uint32_t key1, int32_t bits, const RowsOut& o, hipStream_t stream)
{
#define UQ_LAUNCH_SMALL_(ROWS, MULTI, BITS)                                                                        \
    hipLaunchKernelGGL((k_step_small<ROWS, MULTI, BITS>), dim3(1), dim3(kSmallThreads), 0, stream, g, d, M, ldg,   \
                       w, S, key0, key1, o)
#define UQ_LAUNCH_SMALL(ROWS, MULTI)                                      \
    do {                                                                  \
        if (bits == 8)                                                    \
            UQ_LAUNCH_SMALL_(ROWS, MULTI, 8);                             \
        else if (bits == 4)                                               \
            UQ_LAUNCH_SMALL_(ROWS, MULTI, 4);                             \
        else if (bits == 2)                                               \
            UQ_LAUNCH_SMALL_(ROWS, MULTI, 2);                             \
        else                                                              \
            UQ_LAUNCH_SMALL_(ROWS, MULTI, 0);                             \
    } while (0)
    if (M <= 8) {
        if (S.K > 1) UQ_LAUNCH_SMALL(8, true); else UQ_LAUNCH_SMALL(8, false);
    } else {
        if (S.K > 1) UQ_LAUNCH_SMALL(16, true); else UQ_LAUNCH_SMALL(16, false);
    }
#undef UQ_LAUNCH_SMALL
#undef UQ_LAUNCH_SMALL_
    return hipGetLastError();
}

hipError_t launch_aggregate(const float* g, int64_t d, int32_t M, int64_t ldg, const ScaleSet& S, uint64_t seed,
                            int32_t bits, float* w, uint8_t* idx, uint8_t* codes, int64_t ldc, int32_t* sum,
                            float* out, void* ws, hipStream_t stream)
{
    const uint32_t key0 = static_cast<uint32_t>(seed);
    const uint32_t key1 = static_cast<uint32_t>(seed >> 32);
    const RowsOut o{S.K > 1 ? idx : nullptr, codes, ldc, sum, out};
    const NormPlan plan = norm_plan(d);
    if (d > 0 && d <= small_step(M))
        return launch_step_small(g, d, M, ldg, w, S, key0, key1, bits, o, stream);
    // one scale with codes stored: beyond what the cache holds, summing them
    // as they are stored saves reading them back; below, the quantiser and
    // the sum are faster apart (one scale needs no row of another's):
    // 8 rows of 25.6 M 297 against 311 us at 2 bits, 332 against 349 at 8;
    // 16 rows of 60 M 1554 against 1467 us at 8 bits; with at most kOwnChunks
    // partials a row (but too many for every wave to reduce) that is so from 13
    // rows, where the pass has two waves a SIMD: 16 rows of 2^20, 8 bits 40.8 us
    // against 35.0, 12 rows of 0.8 M 24.4 against 25.6
    const bool own = d > 0 && plan.nchunks <= kOwnChunks && M * plan.nchunks <= kOwnNormPartials;
    const bool apart = bits != 0 && S.K == 1 && d > 0 && !own && (plan.nchunks > kOwnChunks || M > 12) &&
                       static_cast<int64_t>(M) * ((d * bits + 7) / 8) <= kThroughNontemporalBytes;
    double* part = static_cast<double*>(ws);
    const hipError_t e = launch_norm(g, d, M, ldg, plan, own ? nullptr : w, part, stream);
    if (e != hipSuccess || d == 0)
        return e;
    if (apart) {
        const hipError_t q = launch_quantise(g, d, M, ldg, 0, w, S, nullptr, seed, codes, ldc, bits, stream);
        return q != hipSuccess ? q : launch_sum_dequant(codes, d, M, ldc, bits, 0, sum, M, w, S, nullptr, out, stream);
    }
    // one row of one scale: the rows pass codes rows in pairs and would draw a
    // second row's blocks for nothing; the one-row form (512-coordinate tiles)
    // draws each once: 11.2 M coordinates 30.1 us against 33.9, 25.6 M 60.5
    // against 72.9, the same at 3.0 M and below
    if (bits == 0 && S.K == 1 && M == 1 && !own)
        return launch_quant_sum(g, d, 1, ldg, 0, w, S, nullptr, seed, 0, sum, 1, out, stream, 8);
    const WSource src{w, own ? part : nullptr, plan.nchunks};
    if (bits != 0)
        return launch_stored_from(g, d, M, ldg, src, S, key0, key1, bits, o, stream);
    if (S.K > 1)
        return launch_index_quant_sum_from(g, d, M, ldg, src, S, key0, key1, o, stream);
    return launch_quant_sum_split(g, d, M, ldg, 0, src, S, key0, key1, M, o, stream);
}

hipError_t launch_sum(const int8_t* codes, int64_t d, int32_t rows, int64_t ldc, int32_t accumulate,
                      int32_t* sum, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    const unsigned gx = one_shot(d, kSumTile);
    hipLaunchKernelGGL((k_sum<8, 0>), dim3(gx), dim3(kBlock), 0, stream, reinterpret_cast<const uint8_t*>(codes),
                       d, rows, ldc, accumulate, sum, DeqArgs{});
    return hipGetLastError();
}

hipError_t launch_sum_packed(const uint8_t* packed, int64_t d, int32_t rows, int64_t ldp, int32_t bits,
                             int32_t accumulate, int32_t* sum, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    const unsigned gx = one_shot(d, kSumTile);
    if (bits == 4)
        hipLaunchKernelGGL((k_sum<4, 0>), dim3(gx), dim3(kBlock), 0, stream, packed, d, rows, ldp, accumulate, sum,
                           DeqArgs{});
    else
        hipLaunchKernelGGL((k_sum<2, 0>), dim3(gx), dim3(kBlock), 0, stream, packed, d, rows, ldp, accumulate, sum,
                           DeqArgs{});
    return hipGetLastError();
}

hipError_t launch_sum_dequant(const uint8_t* codes, int64_t d, int32_t rows, int64_t ldc, int32_t bits,
                              int32_t accumulate, int32_t* sum, int32_t M, const float* w, const ScaleSet& S,
                              const uint8_t* idx, float* out, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    const unsigned gx = one_shot(d, kSumTile);
    const DeqArgs da{w, idx, out, S, M, 4 * d > kSumNontemporalBytes ? 1 : 0};
#define UQ_LAUNCH_SUM_DEQ(BITS, DEQ)                                                                               \
    hipLaunchKernelGGL((k_sum<BITS, DEQ>), dim3(gx), dim3(kBlock), 0, stream, codes, d, rows, ldc, accumulate, sum, \
                       da)
    const bool multi = S.K > 1;
    if (bits == 8) {
        if (multi) UQ_LAUNCH_SUM_DEQ(8, 2); else UQ_LAUNCH_SUM_DEQ(8, 1);
    } else if (bits == 4) {
        if (multi) UQ_LAUNCH_SUM_DEQ(4, 2); else UQ_LAUNCH_SUM_DEQ(4, 1);
    } else {
        if (multi) UQ_LAUNCH_SUM_DEQ(2, 2); else UQ_LAUNCH_SUM_DEQ(2, 1);
    }
#undef UQ_LAUNCH_SUM_DEQ
    return hipGetLastError();
}

hipError_t launch_dequant(const int32_t* sum, int64_t d, int32_t M, const float* w, const ScaleSet& S,
                          const uint8_t* idx, float* out, hipStream_t stream)
{
    if (d == 0)
        return hipSuccess;
    const int64_t tile = 256 * dequant_quads(S.K > 1);
    const int64_t ntiles = (d + tile - 1) / tile;
    const int64_t cap = one_shot_cap();
    for (int64_t tile0 = 0; tile0 < ntiles; tile0 += cap) {
        const dim3 grid(blocks_from(ntiles, tile0, cap));
#define UQ_LAUNCH_DEQUANT(MULTI, NT) \
    hipLaunchKernelGGL((k_dequant<MULTI, NT>), grid, dim3(64), 0, stream, sum, d, M, w, S, idx, tile0, out)
        const bool nt = 4 * d > kSumNontemporalBytes;
        if (S.K > 1) {
            if (nt) UQ_LAUNCH_DEQUANT(true, true); else UQ_LAUNCH_DEQUANT(true, false);
        } else {
            if (nt) UQ_LAUNCH_DEQUANT(false, true); else UQ_LAUNCH_DEQUANT(false, false);
        }
#undef UQ_LAUNCH_DEQUANT
    }
    return hipGetLastError();
}

}  // namespace uq
