// fp32 module on v_mfma_f32_16x16x4_f32 (fp32 products and sums, no narrower type anywhere).  f32_kernel takes the products of the
// forward and backward (x W^T, x A^T, h B^T, dz B, dz W + dh A, dh^T x, dz^T h) and A A^T where it is asked for, up to three of
// them and dm's column sum in a launch; norm_f32_kernel the row norm.  An operand is row-major [rows, K] (K-contiguous) or
// row-major [K, rows] (K-strided), its row stride and the extent of its contiguous axis multiples of four elements.
//
// A lane (m = lane & 15, q = lane >> 4) of the MFMA supplies one k.  Both operands take k = 4 q + j for the j-th of four
// MFMAs, so a lane's four k of a group of 16 are consecutive: one 16-byte read of a K-contiguous row.
//
// Rows past the end are clamped to the last one (they only reach outputs that are not stored); k past the end is set to
// zero on both sides, by selection, so that a NaN or infinity in a neighbouring row is not multiplied in.
//
// Bound: launches and the latency of a chain of loads for small modules, the matrix cores (157 TFLOP/s) and the last round of
// tiles for larger ones.  Forward and backward of 256 x 512, r 16, 64 tokens take five launches, 29 us (eleven, one for each
// product and pass, 49), of 1000 x 772, r 36, 1500 tokens 118 us (171), of 256 x 512, r 64, 8192 tokens 167 (196), of 4096 x 4096,
// r 384, 2048 tokens 1950 (2070); 43 shapes 1.02 to 1.84 times faster than the eleven.
#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace dora {
namespace {

__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// elements k .. k+3 of row `row` (clamped) of an operand with `rows` rows and K k's; zeros where k is past the end
template <bool KC>
__device__ __forceinline__ float4 load_k4(const float* __restrict__ p, int64_t ld, int rows, int K, int row, int k)
{
    const int rr = row < rows ? row : rows - 1;
    float4 v;
    if constexpr (KC) {
        const int kk = k < K ? k : K - 4;              // K is a multiple of four
        v = *reinterpret_cast<const float4*>(p + (int64_t)rr * ld + kk);
        if (k >= K) v = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        float e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kk = k + j < K ? k + j : K - 1;
            e[j] = p[(int64_t)kk * ld + rr];
        }
        v = make_float4(k < K ? e[0] : 0.f, k + 1 < K ? e[1] : 0.f, k + 2 < K ? e[2] : 0.f, k + 3 < K ? e[3] : 0.f);
    }
    return v;
}

__device__ __forceinline__ float get(const float4& v, int j) { return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w; }

__device__ __forceinline__ float4 mul4(const float4& a, const float4& b) { return make_float4(a.x * b.x, a.y * b.y, a.z * b.z, a.w * b.w); }

__device__ __forceinline__ float scale_of(const RowScale& s, int i)
{
    const float v = s.g[i];
    if (!s.m) return v;
    const float cc = (v < s.eps) ? s.eps : v;          // NaN stays NaN
    return s.m[i] / cc;
}
// What becomes of four elements of a row of the product (N, ldc and the pointers' alignment allow whole vectors).
__device__ __forceinline__ void finish(const SgemmArgs& p, int m, int n, float4 v)
{
    float4* const c = reinterpret_cast<float4*>(p.c + (int64_t)m * p.ldc + n);
    v = make_float4(p.alpha * v.x, p.alpha * v.y, p.alpha * v.z, p.alpha * v.w);
    if (p.composed) {                                  // as the compose pass: s lora first, then g (.)
        const float4 b = *c, g = *reinterpret_cast<const float4*>(p.g + n), g1 = *reinterpret_cast<const float4*>(p.gm1 + n);
        float4 bias = make_float4(0.f, 0.f, 0.f, 0.f), y, in;
        if (p.bias) bias = *reinterpret_cast<const float4*>(p.bias + n);
        auto one = [&](float bv, float gv, float g1v, float lora, float add, float& yv, float& iv) {
            const float sl = p.s * lora, delta = fmaf(g1v, bv, gv * sl);
            yv = (bv + delta) + add;
            iv = sl + bv;
        };
        one(b.x, g.x, g1.x, v.x, bias.x, y.x, in.x);
        one(b.y, g.y, g1.y, v.y, bias.y, y.y, in.y);
        one(b.z, g.z, g1.z, v.z, bias.z, y.z, in.z);
        one(b.w, g.w, g1.w, v.w, bias.w, y.w, in.w);
        *c = y;
        if (p.inner) *reinterpret_cast<float4*>(p.inner + (int64_t)m * p.ldc + n) = in;
    } else {
        if (p.rowscale.g) {
            const float f = scale_of(p.rowscale, m);
            v = make_float4(f * v.x, f * v.y, f * v.z, f * v.w);
        }
        *c = v;
    }
}

// Few tiles: 32 x 32 of C per workgroup, its WK waves split K and meet in LDS at the end.  These products are bound by
// the latency of a serial K loop, not by arithmetic, so the fragments come straight from memory into registers, DEPTH
// groups of 16 k in flight per wave, and no wave waits for another before the end.
constexpr int SPLIT_LD = 36;
template <int WK, bool SHORT, bool A_KC, bool B_KC>
__device__ __forceinline__ void split_product(const SgemmArgs& p, int wg, float* red)
{
    constexpr bool MAY_SCALE = A_KC && !B_KC;
    constexpr int DEPTH = 4, LD = SPLIT_LD;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int M = p.M, N = p.N;
    const int tiles_n = (N + 31) / 32;                 // one-dimensional grid: no 65535 limit on the row-tile count
    const int m0 = wg / tiles_n * 32, n0 = wg % tiles_n * 32;
    // SHORT: a sum of its own for every 64 k of a wave.  As one chain of additions a wave's share of K has up to twice the error (four
    // waves, 704 x 1760, r 20, 1509 tokens, dB 5.2e-7, in short sums 2.3e-7; sixteen, 64 x 64, r 4, 20000 tokens 7.2e-7 and 2.4e-7).
    // Four waves always take them, sixteen (3 % slower with them over a K of 10000) where they stand in for four.
    f32x4_t acc[2][2], total[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = total[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int sidx = 0; sidx < p.nseg; ++sidx) {
        const SgemmSeg sg = p.seg[sidx];
        const bool scaled = MAY_SCALE && sg.scaled;
        const int groups = (sg.K + 15) / 16;
        const int g_begin = (int)((int64_t)groups * wave / WK), g_end = (int)((int64_t)groups * (wave + 1) / WK);
        for (int g = g_begin; g < g_end; g += DEPTH) {
            float4 a[DEPTH][2], b[DEPTH][2];
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (g + d < g_end) {
                    const int k = (g + d) * 16 + lq * 4;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        a[d][i] = load_k4<A_KC>(sg.a, sg.lda, M, sg.K, m0 + i * 16 + l16, k);
                        b[d][i] = load_k4<B_KC>(sg.b, sg.ldb, N, sg.K, n0 + i * 16 + l16, k);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) a[d][i] = b[d][i] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
            // the scales of these 64 k, one to a lane, pass through this wave's part of `red` (zero past the end)
            float* const mine = red + wave * 32 * LD;
            if (scaled) {
                const int k = g * 16 + lane;
                mine[lane] = k < sg.K ? scale_of(p.ascale, k) : 0.f;
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (g + d < g_end) {
                    if (scaled) {
                        const float4 f = *reinterpret_cast<const float4*>(mine + d * 16 + lq * 4);
#pragma unroll
                        for (int i = 0; i < 2; ++i) a[d][i] = mul4(a[d][i], f);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(get(b[d][j], e), get(a[d][i], e), acc[i][j]);
                }
            if (scaled) __builtin_amdgcn_wave_barrier();
            if constexpr (SHORT) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        total[i][j] += acc[i][j];
                        acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
    }
    // lane: columns 4 lq .. +3 of block j, row l16 of block i
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<f32x4_t*>(red + wave * 32 * LD + (i * 16 + l16) * LD + j * 16 + lq * 4) = SHORT ? total[i][j] : acc[i][j];
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += 64 * WK) {
        const int m = e / 8, n = e % 8 * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < WK; ++w) {
            const float4 u = *reinterpret_cast<const float4*>(red + w * 32 * LD + m * LD + n);
            v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        if (m0 + m < M && n0 + n < N) finish(p, m0 + m, n0 + n, v);
    }
}

// LDS offset (floats) of the 16-byte chunk `c` (four k) of row `row` in a [.][32] tile of the kernel below: rows of 128
// bytes, chunks XORed so that the 16 rows of a fragment read cover all 16 slots of 256 bytes, and so that the rows 4 apart
// which a wave turns around on the way in do as well as rows of one parity can (two lanes a slot).
__device__ __forceinline__ int tile_off(int row, int c) { return row * 32 + ((c ^ (row >> 1) ^ (row >> 4)) & 7) * 4; }

// Many tiles: TM x 64 of C per workgroup, TM / 2 x 32 per wave, K in steps of 32 through two LDS buffers.  One or two
// workgroups per CU do not hide a load's latency, so steps are fetched into registers two ahead; a K-strided operand is
// turned around, 4 x 4 elements per thread, on the way into LDS.  (One step ahead and rows padded to 144 bytes: dz W + dh A of
// 1500 x 772 x 1036 in 76 us; 56 with 64-row tiles, 53 with 32-row ones and dA and dB in the same launch.)
constexpr int TS = 64, TK = 32;
template <int TM, bool A_KC, bool B_KC>
__device__ __forceinline__ void tile_product(const SgemmArgs& p, int wg, float* lds_)
{
    constexpr int MT = TM / 32;                        // blocks of 16 rows per wave
    constexpr bool MAY_SCALE = A_KC && !B_KC;
    float (*const lds)[2][TS * TK] = reinterpret_cast<float (*)[2][TS * TK]>(lds_);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int M = p.M, N = p.N;
    const int tiles_n = (N + TS - 1) / TS;
    const int m0 = wg / tiles_n * TM, n0 = wg % tiles_n * TS;
    const int wm0 = wave / 2 * (TM / 2), wn0 = wave % 2 * 32;
    // threads 0..127 bring in the M-side operand, the others the N-side one, up to 16 elements of a step each: k 4 kg .. +3 of
    // rows rg, rg + 16, .. (K-contiguous) or rows 4 rg .. +3 of k 4 kg .. +3 (K-strided)
    const bool n_side = wave >= 2;
    const bool kc = n_side ? B_KC : A_KC;
    const int blk = tid & 127, side = n_side ? TS : TM;
    const int rg = kc ? blk / (TK / 4) : blk % (side / 4), kg = kc ? blk % (TK / 4) : blk / (side / 4);
    const int vecs = kc ? side / 16 : kg < TK / 4 ? 4 : 0;
    const int row0 = (n_side ? n0 : m0) + (kc ? rg : rg * 4), rows = n_side ? N : M;
    f32x4_t acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int sidx = 0; sidx < p.nseg; ++sidx) {
        const SgemmSeg sg = p.seg[sidx];
        const float* const base = n_side ? sg.b : sg.a;
        const int64_t ld = n_side ? sg.ldb : sg.lda;
        const int K = sg.K, steps = (K + TK - 1) / TK;
        // (the scale as it is: the launch before this one formed it)
        const bool scaled = MAY_SCALE && sg.scaled && !n_side;
        auto fetch = [&](int step, float4 (&v)[MAY_SCALE ? 5 : 4]) {
            const int k = step * TK + kg * 4;
            if constexpr (MAY_SCALE) v[4] = scaled ? *reinterpret_cast<const float4*>(p.ascale.g + (k < K ? k : K - 4)) : make_float4(1.f, 1.f, 1.f, 1.f);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (TM < TS && i >= vecs) continue;
                if (kc) {
                    const int row = row0 + 16 * i;
                    const int rr = row < rows ? row : rows - 1, kk = k < K ? k : K - 4;
                    v[i] = *reinterpret_cast<const float4*>(base + (int64_t)rr * ld + kk);
                } else {                               // rows is a multiple of four
                    const int rr = row0 < rows ? row0 : rows - 4, kk = k + i < K ? k + i : K - 1;
                    v[i] = *reinterpret_cast<const float4*>(base + (int64_t)kk * ld + rr);
                }
            }
        };
        auto stage = [&](int step, const float4 (&v)[MAY_SCALE ? 5 : 4]) {
            float* const tile = lds[step & 1][n_side];
            const int k = step * TK + kg * 4;
            float4 w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (MAY_SCALE) w[i] = mul4(v[i], v[4]);   // only where K is the contiguous axis: all four of one k each
                else w[i] = v[i];
                if (k + (kc ? 0 : i) >= K) w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (TM < TS && i >= vecs) continue;
                if (kc) *reinterpret_cast<float4*>(tile + tile_off(rg + 16 * i, kg)) = w[i];
                else *reinterpret_cast<float4*>(tile + tile_off(rg * 4 + i, kg)) =
                         make_float4(get(w[0], i), get(w[1], i), get(w[2], i), get(w[3], i));
            }
        };
        // step t from LDS; `next` holds step t + 1 (staged at the end), `far` takes step t + 2
        auto body = [&](int t, const float4 (&next)[MAY_SCALE ? 5 : 4], float4 (&far)[MAY_SCALE ? 5 : 4]) {
            if (t + 2 < steps) fetch(t + 2, far);
            const float* const as = lds[t & 1][0];
            const float* const bs = lds[t & 1][1];
#pragma unroll
            for (int q = 0; q < TK / 16; ++q) {
                float4 a[MT], b[2];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const float4*>(as + tile_off(wm0 + i * 16 + l16, q * 4 + lq));
#pragma unroll
                for (int i = 0; i < 2; ++i) b[i] = *reinterpret_cast<const float4*>(bs + tile_off(wn0 + i * 16 + l16, q * 4 + lq));
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(get(b[j], e), get(a[i], e), acc[i][j]);
            }
            if (t + 1 < steps) stage(t + 1, next);     // that buffer was read last in step t - 1, before its barrier
            __syncthreads();
        };
        float4 va[MAY_SCALE ? 5 : 4], vb[MAY_SCALE ? 5 : 4];
        if (steps > 0) { fetch(0, va); stage(0, va); }
        if (steps > 1) fetch(1, vb);
        __syncthreads();
        for (int t = 0; t < steps; t += 2) {
            body(t, vb, va);
            if (t + 1 < steps) body(t + 1, va, vb);
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = m0 + wm0 + i * 16 + l16;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn0 + j * 16 + lq * 4;
            if (n < N) finish(p, m, n, make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]));
        }
    }
}

// First stage of dm's column sum: 256 columns of COLUMN_SUM_ROWS tokens, a float4 per lane.  Sixteen sums take rows in turn and are
// added in order, 16 / WK of them to a wave, so that dm does not depend on how many waves the launch has.
constexpr int SUMS = 16;
template <int WK>
__device__ __forceinline__ void column_sum(const ColumnSum& p, int wg, float* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col_blocks = (p.d_out + 255) / 256, slab = wg / col_blocks, col = (wg % col_blocks) * 256 + lane * 4;
    const int64_t row0 = (int64_t)slab * COLUMN_SUM_ROWS;
    for (int q = wave; q < SUMS; q += WK) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (col < p.d_out) {
            constexpr int U = COLUMN_SUM_ROWS / SUMS;
            float4 d[U], n[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t row = row0 + q + u * SUMS, at = (row < p.tokens ? row : p.tokens - 1) * p.d_out + col;
                d[u] = *reinterpret_cast<const float4*>(p.dy + at);
                n[u] = *reinterpret_cast<const float4*>(p.inner + at);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (row0 + q + u * SUMS < p.tokens) {
                    acc.x = fmaf(d[u].x, n[u].x, acc.x); acc.y = fmaf(d[u].y, n[u].y, acc.y);
                    acc.z = fmaf(d[u].z, n[u].z, acc.z); acc.w = fmaf(d[u].w, n[u].w, acc.w);
                }
        }
        *reinterpret_cast<float4*>(red + q * 256 + lane * 4) = acc;
    }
    __syncthreads();
    const int j = (wg % col_blocks) * 256 + (int)threadIdx.x;
    if (threadIdx.x < 256 && j < p.d_out) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < SUMS; ++w) v += red[w * 256 + threadIdx.x];
        p.partial[(int64_t)slab * p.d_out + j] = v;
    }
}

// Second stage: 64 columns per workgroup, sixteen sums take slabs in turn.
template <int WK>
__device__ __forceinline__ void column_final(const ColumnFinal& p, int wg, float* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = wg * 64 + lane;
    constexpr int PER = SUMS / WK, U = PER == 1 ? 4 : 2;
    float v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) v[q] = 0.f;
    if (j < p.d_out)
        for (int z = 0; z < p.slabs; z += U * SUMS) {
            float e[PER][U];
#pragma unroll
            for (int q = 0; q < PER; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int at = z + u * SUMS + wave * PER + q;
                    e[q][u] = p.partial[(int64_t)(at < p.slabs ? at : p.slabs - 1) * p.d_out + j];
                }
#pragma unroll
            for (int q = 0; q < PER; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u) v[q] += z + u * SUMS + wave * PER + q < p.slabs ? e[q][u] : 0.f;
        }
#pragma unroll
    for (int q = 0; q < PER; ++q) red[(wave * PER + q) * 64 + lane] = v[q];
    __syncthreads();
    if (wave == 0 && j < p.d_out) {
        float sum = red[lane];
        for (int w = 1; w < SUMS; ++w) sum += red[w * 64 + lane];
        const float cc = (p.c[j] < p.eps) ? p.eps : p.c[j];
        p.dm[j] = sum / cc;
    }
}

// One launch of several pieces of work that do not need one another: the small module's products are a few microseconds each,
// most of it launch and latency.  Workgroups below first[0] do piece 0, and so on.
struct F32Launch {
    SgemmArgs g[3];
    ColumnSum sum;
    ColumnFinal fin;
    ScaleOut scale;
    int first[5];            // ends of the products' workgroups, of the column sum's two stages, of the scale's
    int tiled[3];            // rows of a tile: 64 x 64 or 32 x 64, or 0: split 32 x 32 ones
};

template <int WK, bool SHORT>
__global__ __launch_bounds__(64 * WK, 4) void f32_kernel(F32Launch p)
{
    constexpr int FLOATS = WK * 32 * SPLIT_LD > 2 * 2 * TS * TK ? WK * 32 * SPLIT_LD : 2 * 2 * TS * TK;
    __shared__ __attribute__((aligned(256))) float lds[FLOATS];
    const int id = blockIdx.x;
    if (id >= p.first[4]) {
        const int j = (id - p.first[4]) * 64 * WK + (int)threadIdx.x;
        if (j < p.scale.n) p.scale.out[j] = scale_of(p.scale.scale, j);
        return;
    }
    if (id >= p.first[3]) return column_final<WK>(p.fin, id - p.first[3], lds);
    if (id >= p.first[2]) return column_sum<WK>(p.sum, id - p.first[2], lds);
    const int q = id < p.first[0] ? 0 : id < p.first[1] ? 1 : 2, wg = id - (q == 0 ? 0 : p.first[q - 1]);
    const SgemmArgs& g = p.g[q];
    if constexpr (WK == 4) {
        auto tile = [&](auto rows) {
            constexpr int TM = decltype(rows)::value;
            if (!g.a_kcontig) tile_product<TM, false, false>(g, wg, lds);
            else if (g.b_kcontig) tile_product<TM, true, true>(g, wg, lds);
            else tile_product<TM, true, false>(g, wg, lds);
        };
        if (p.tiled[q] == 64) return tile(std::integral_constant<int, 64>{});
        if (p.tiled[q] == 32) return tile(std::integral_constant<int, 32>{});
    }
    if (!g.a_kcontig) split_product<WK, SHORT, false, false>(g, wg, lds);
    else if (g.b_kcontig) split_product<WK, SHORT, true, true>(g, wg, lds);
    else split_product<WK, SHORT, true, false>(g, wg, lds);
}

int64_t tiles(const SgemmArgs& a, int tm, int tn) { return a.M <= 0 || a.N <= 0 ? 0 : (int64_t)((a.N + tn - 1) / tn) * ((a.M + tm - 1) / tm); }

int longest_k(const SgemmArgs& a) { return a.nseg > 1 && a.seg[1].K > a.seg[0].K ? a.seg[1].K : a.seg[0].K; }

// Tiles once 64 x 64 ones fill half the chip; below, the split ones (0).  32 x 64 where they share the CUs out better: half
// the work a tile at nine tenths of the rate.
int tile_rows(const SgemmArgs& a)
{
    const int64_t t64 = tiles(a, 64, TS), t32 = tiles(a, 32, TS);
    if (t64 < 128) return 0;
    return (t32 + 255) / 256 * 11 < (t64 + 255) / 256 * 20 ? 32 : 64;
}

int64_t sum_of_k(const SgemmArgs& a) { return a.seg[0].K + (a.nseg > 1 ? (int64_t)a.seg[1].K : 0); }

// Time of a workgroup in tenths of a microsecond: 5 for a step of 32 k in tiles, 10 for 256 k of a split product in four waves.
int64_t wg_cost(const SgemmArgs& a) { return tile_rows(a) ? sum_of_k(a) / 32 * 5 : sum_of_k(a) / 256 * 10; }

// Beside tiles a split product has four waves to a workgroup instead of sixteen.  Where its K is so long that it would end well
// after the tiles (steps of 32 k: a CU's share of them, or a tile's own), it goes to a launch of its own.  (Backward, in one launch
// and in two: 84 x 12, r 4, 29613 tokens 329 us and 253; 14876 x 548, r 20, 2 tokens 292 and 235; 8 x 464, r 20, 20141 tokens 229
// and 198; 56 x 900, r 44, 666 tokens 15.5 and 23; 76 x 3904, r 16, 1180 tokens 36 and 44.  Over 200 mixed shapes the line is
// within 0.1 % of always taking the faster one; always one launch 3.5 %, always two 9.7 %.)
bool split_apart(const SgemmArgs* g, int n)
{
    int64_t share = 0, longest = 0, k = 0;
    for (int i = 0; i < n; ++i) {
        if (g[i].M <= 0 || g[i].N <= 0) continue;
        const int64_t steps = (sum_of_k(g[i]) + 31) / 32;
        if (tile_rows(g[i])) { share += tiles(g[i], 64, TS) * steps; longest = std::max(longest, steps); }
        else k = std::max(k, sum_of_k(g[i]));
    }
    return share > 0 && k > 1000 + 400 * std::max(share / 256, longest);
}

hipError_t launch_one(const SgemmArgs* g, int n, const ColumnSum* sum, const ColumnFinal* fin, const ScaleOut* scale, int trace_id,
                      hipStream_t stream, bool short_sums)
{
    F32Launch p{};
    int64_t end = 0;
    bool any_tiled = false, long_k = false;
    for (int i = 0; i < n; ++i) {
        if (!g[i].a_kcontig && g[i].b_kcontig) return hipErrorInvalidValue;
        const int rows = tile_rows(g[i]);
        // a scale in tiles is taken as it is: one that has to be formed there would pass as its own denominator
        for (int k = 0; k < g[i].nseg; ++k)
            if (rows && g[i].seg[k].scaled && g[i].ascale.m) return hipErrorInvalidValue;
        any_tiled |= rows != 0;
        long_k |= longest_k(g[i]) >= 256;
        // the one whose workgroups take longest first: a split one of many k behind rounds of tiles would end alone
        int at = i;
        for (; at > 0 && wg_cost(g[i]) > wg_cost(p.g[at - 1]); --at) { p.g[at] = p.g[at - 1]; p.tiled[at] = p.tiled[at - 1]; }
        p.g[at] = g[i];
        p.tiled[at] = rows;
    }
    for (int i = 0; i < 3; ++i) {
        if (i < n) end += p.tiled[i] ? tiles(p.g[i], p.tiled[i], TS) : tiles(p.g[i], 32, 32);
        p.first[i] = (int)end;
    }
    if (sum) { p.sum = *sum; end += (int64_t)((sum->d_out + 255) / 256) * column_sum_slabs(sum->tokens); }
    p.first[3] = (int)end;
    if (fin) { p.fin = *fin; end += (fin->d_out + 63) / 64; }
    p.first[4] = (int)end;
    const bool sixteen = long_k && !any_tiled;
    if (scale) { p.scale = *scale; end += (scale->n + (sixteen ? 1023 : 255)) / (sixteen ? 1024 : 256); }
    if (end == 0) return hipSuccess;
    TraceScope ts(trace_id, stream);
    // sixteen waves to a workgroup where a product's K gives each of them a group of 16, four beside tiles and for the
    // products over the rank
    if (sixteen && short_sums) f32_kernel<16, true><<<dim3((unsigned)end), dim3(64 * 16), 0, stream>>>(p);
    else if (sixteen) f32_kernel<16, false><<<dim3((unsigned)end), dim3(64 * 16), 0, stream>>>(p);
    else f32_kernel<4, true><<<dim3((unsigned)end), dim3(64 * 4), 0, stream>>>(p);
    return hipGetLastError();
}

// Norm: 16 or 32 rows per workgroup, its sixteen waves take 32 columns in turn.  V = B A of those stays in registers and meets W
// there; the three sums of Eq. 2 of whole rows end in one workgroup, which finishes Eq. 5 and 6.  Where few rows leave CUs without
// one, or a round of workgroups is badly filled, the columns are cut into slices and the sums go to memory.  Bound by the
// matrix cores (8192 x 8192, r 384 at 87 TFLOP/s of 157) and, with 16 rows, by reading A from the L2 (72).  (U = W A^T, A A^T, B G
// and the row sums as four pieces of work in three launches: 1000 x 772, r 36 17 us, this one 10; 2048 x 2048, r 128 61, 22; 8192 x
// 8192, r 384 646, 595; 27648 x 5120, r 384 1352, 1323; error against 64 bits 4.7e-8, 4.4e-8.)
constexpr int NORM_WAVES = 16;
template <int RB>   // blocks of 16 rows
__global__ __launch_bounds__(64 * NORM_WAVES) void norm_f32_kernel(NormF32Args p)
{
    constexpr int DEPTH = 4 / RB, ROWS = 16 * RB;
    __shared__ float red[NORM_WAVES][3][ROWS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int slice = blockIdx.x % p.slices, m0 = blockIdx.x / p.slices * ROWS;
    const int d_in = p.d_in, r = p.r, groups = (r + 15) / 16;
    int row[RB];
    float sum[RB][3];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int m = m0 + i * 16 + l16;
        row[i] = m < p.d_out ? m : p.d_out - 1;
        sum[i][0] = sum[i][1] = sum[i][2] = 0.f;
    }
    for (int n0 = (wave * p.slices + slice) * 32; n0 < d_in; n0 += p.slices * NORM_WAVES * 32) {
        float4 w[RB][2];
        f32x4_t acc[RB][2];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + j * 16 + lq * 4;
                w[i][j] = *reinterpret_cast<const float4*>(p.w + (int64_t)row[i] * d_in + (n < d_in ? n : d_in - 4));
                acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        for (int g = 0; g < groups; g += DEPTH) {
            float4 b[DEPTH][RB], a[DEPTH][2];
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {          // groups past the end bring zeros
                const int k = (g + d) * 16 + lq * 4;
#pragma unroll
                for (int i = 0; i < RB; ++i) b[d][i] = load_k4<true>(p.b, r, p.d_out, r, row[i], k);
#pragma unroll
                for (int j = 0; j < 2; ++j) a[d][j] = load_k4<false>(p.a, d_in, d_in, r, n0 + j * 16 + l16, k);
            }
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (g + d < groups)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = 0; i < RB; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(get(a[d][j], e), get(b[d][i], e), acc[i][j]);
        }
        // lane: columns 4 lq .. +3 of block j, row l16 of block i
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (n0 + j * 16 + lq * 4 < d_in)
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    float t[3] = {0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float wv = get(w[i][j], e), v = acc[i][j][e];
                        t[0] = fmaf(wv, wv, t[0]); t[1] = fmaf(wv, v, t[1]); t[2] = fmaf(v, v, t[2]);
                    }
#pragma unroll
                    for (int k = 0; k < 3; ++k) sum[i][k] += t[k];
                }
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            sum[i][k] += __shfl_xor(sum[i][k], 16);
            sum[i][k] += __shfl_xor(sum[i][k], 32);
            if (lq == 0) red[wave][k][i * 16 + l16] = sum[i][k];
        }
    __syncthreads();
    const int j = m0 + (int)threadIdx.x;
    if (threadIdx.x >= ROWS || j >= p.d_out) return;
    float all[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double v = 0.;
#pragma unroll
        for (int i = 0; i < NORM_WAVES; ++i) v += red[i][k][threadIdx.x];
        all[k] = (float)v;
    }
    if (p.slices > 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) p.part[((int64_t)k * p.slices + slice) * p.d_out + j] = all[k];
        return;
    }
    if (p.base_in) all[0] = p.base_in[j];
    if (p.terms)
#pragma unroll
        for (int k = 0; k < 3; ++k) p.terms[(int64_t)k * p.d_out + j] = all[k];
    if (!p.c) return;
    const float cj = __fsqrt_rn(radicand(all[0], all[1], all[2], p.two_s, p.s2));
    p.c[j] = cj;
    if (p.m) {
        const float cc = (cj < p.eps) ? p.eps : cj, mj = p.m[j];
        if (p.g) p.g[j] = mj / cc;
        if (p.gm1) p.gm1[j] = (mj - cc) / cc;
    }
}

}  // namespace

bool f32_tiled(const SgemmArgs& a) { return tile_rows(a) != 0; }

hipError_t launch_f32(const SgemmArgs* g, int n, const ColumnSum* sum, const ColumnFinal* fin, const ScaleOut* scale,
                      int trace_id, hipStream_t stream)
{
    if (n < 0 || n > 3) return hipErrorInvalidValue;
    if (!split_apart(g, n)) return launch_one(g, n, sum, fin, scale, trace_id, stream, false);
    SgemmArgs part[2][3];
    int m[2] = {0, 0};
    for (int i = 0; i < n; ++i) {
        const int t = tile_rows(g[i]) != 0;
        part[t][m[t]++] = g[i];
    }
    const hipError_t e = launch_one(part[0], m[0], sum, fin, scale, trace_id, stream, true);
    return e != hipSuccess ? e : launch_one(part[1], m[1], nullptr, nullptr, nullptr, trace_id, stream, false);
}

hipError_t launch_norm_f32(const NormF32Args& a, hipStream_t stream)
{
    TraceScope ts(DORA_K_NORM_CROSS, stream);
    if (a.row_blocks == 2) norm_f32_kernel<2><<<dim3((unsigned)((a.d_out + 31) / 32 * a.slices)), dim3(64 * NORM_WAVES), 0, stream>>>(a);
    else norm_f32_kernel<1><<<dim3((unsigned)((a.d_out + 15) / 16 * a.slices)), dim3(64 * NORM_WAVES), 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace dora
