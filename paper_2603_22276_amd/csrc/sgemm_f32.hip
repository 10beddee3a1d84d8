// fp32 GEMM of the fp32 configuration of the module, on v_mfma_f32_16x16x4_f32 (fp32 products and sums, no narrower
// type anywhere).  One pair of kernels serves every contraction of the forward and backward (x W^T, x A^T, h B^T, dz B,
// dz W + dh A, dh^T x, dz^T h) and of Algorithm 1 (W A^T, A A^T, B G); an operand is row-major [rows, K] (K-contiguous) or
// row-major [K, rows] (K-strided), its row stride and the extent of its contiguous axis multiples of four elements.
//
// A lane (m = lane & 15, q = lane >> 4) of the MFMA supplies one k.  Both operands take k = 4 q + j for the j-th of four
// MFMAs, so a lane's four k of a group of 16 are consecutive: one 16-byte read of a K-contiguous row.
//
// Rows past the end are clamped to the last one (they only reach outputs that are not stored); k past the end is set to
// zero on both sides, by selection, so that a NaN or infinity in a neighbouring row is not multiplied in.
//
// Against 32 x 32 and 64 x 64 tiles on the vector unit with one serial K loop per workgroup, forward and backward:
// 256 x 512, r 16, 64 tokens 172 -> 49 us; 1000 x 772, r 36, 1500 tokens 569 -> 171 us.
#include "common.hpp"

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

// Few tiles: 32 x 32 of C per workgroup, its WK waves split K and meet in LDS at the end.  These launches are bound by
// the latency of a serial K loop, not by arithmetic, so the fragments come straight from memory into registers, DEPTH
// groups of 16 k in flight per wave, and no wave waits for another before the end.
template <int WK, bool A_KC, bool B_KC>
__global__ __launch_bounds__(64 * WK) void sgemm_split_kernel(SgemmPair grp)
{
    constexpr int DEPTH = 4, LD = 36;
    __shared__ __attribute__((aligned(16))) float red[WK][32 * LD];
    const bool second = (int)blockIdx.x >= grp.count0;
    const SgemmArgs& p = second ? grp.g[1] : grp.g[0];
    const int wg = (int)blockIdx.x - (second ? grp.count0 : 0);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int M = p.M, N = p.N;
    const int tiles_n = (N + 31) / 32;                 // one-dimensional grid: no 65535 limit on the row-tile count
    const int m0 = wg / tiles_n * 32, n0 = wg % tiles_n * 32;
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int sidx = 0; sidx < p.nseg; ++sidx) {
        const SgemmSeg sg = p.seg[sidx];
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
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (g + d < g_end) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(get(b[d][j], e), get(a[d][i], e), acc[i][j]);
                }
        }
    }
    // lane: columns 4 lq .. +3 of block j, row l16 of block i
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<f32x4_t*>(&red[wave][(i * 16 + l16) * LD + j * 16 + lq * 4]) = acc[i][j];
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += 64 * WK) {
        const int m = e / 32, n = e % 32;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WK; ++w) v += red[w][m * LD + n];
        if (m0 + m < M && n0 + n < N) p.c[(int64_t)(m0 + m) * p.ldc + n0 + n] = p.alpha * v;
    }
}

// LDS offset (floats) of the 16-byte chunk `c` (four k) of row `row` in a [64][32] tile of the kernel below: rows of 128
// bytes, chunks XORed so that the 16 rows of a fragment read cover all 16 slots of 256 bytes, and so that the rows 4 apart
// which a wave turns around on the way in do as well as rows of one parity can (two lanes a slot).
__device__ __forceinline__ int tile_off(int row, int c) { return row * 32 + ((c ^ (row >> 1) ^ (row >> 4)) & 7) * 4; }

// Many tiles: 64 x 64 of C per workgroup, 32 x 32 per wave, K in steps of 32 through two LDS buffers.  One or two
// workgroups per CU do not hide a load's latency, so steps are fetched into registers two ahead; a K-strided operand is
// turned around, 4 x 4 elements per thread, on the way into LDS.  (One step ahead and rows padded to 144 bytes: dz W + dh A of
// 1500 x 772 x 1036 in 76 us, 56 now.)
template <bool A_KC, bool B_KC>
__global__ __launch_bounds__(256) void sgemm_tile_kernel(SgemmArgs p)
{
    constexpr int TS = 64, TK = 32;
    __shared__ __attribute__((aligned(256))) float lds[2][2][TS * TK];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int M = p.M, N = p.N;
    const int tiles_n = (N + TS - 1) / TS;
    const int m0 = (int)(blockIdx.x / tiles_n) * TS, n0 = (int)(blockIdx.x % tiles_n) * TS;
    const int wm0 = wave / 2 * 32, wn0 = wave % 2 * 32;
    // threads 0..127 bring in the M-side operand, the others the N-side one, 16 elements of a step each: k 4 kg .. +3 of
    // rows rg, rg + 16, +32, +48 (K-contiguous) or rows 4 rg .. +3 of k 4 kg .. +3 (K-strided)
    const bool n_side = wave >= 2;
    const bool kc = n_side ? B_KC : A_KC;
    const int blk = tid & 127;
    const int rg = kc ? blk / (TK / 4) : blk % (TS / 4), kg = kc ? blk % (TK / 4) : blk / (TS / 4);
    const int row0 = (n_side ? n0 : m0) + (kc ? rg : rg * 4), rows = n_side ? N : M;
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int sidx = 0; sidx < p.nseg; ++sidx) {
        const SgemmSeg sg = p.seg[sidx];
        const float* const base = n_side ? sg.b : sg.a;
        const int64_t ld = n_side ? sg.ldb : sg.lda;
        const int K = sg.K, steps = (K + TK - 1) / TK;
        auto fetch = [&](int step, float4 (&v)[4]) {
            const int k = step * TK + kg * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
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
        auto stage = [&](int step, const float4 (&v)[4]) {
            float* const tile = lds[step & 1][n_side];
            const int k = step * TK + kg * 4;
            float4 w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w[i] = v[i];
                if (k + (kc ? 0 : i) >= K) w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kc) *reinterpret_cast<float4*>(tile + tile_off(rg + 16 * i, kg)) = w[i];
                else *reinterpret_cast<float4*>(tile + tile_off(rg * 4 + i, kg)) =
                         make_float4(get(w[0], i), get(w[1], i), get(w[2], i), get(w[3], i));
            }
        };
        // step t from LDS; `next` holds step t + 1 (staged at the end), `far` takes step t + 2
        auto body = [&](int t, const float4 (&next)[4], float4 (&far)[4]) {
            if (t + 2 < steps) fetch(t + 2, far);
            const float* const as = lds[t & 1][0];
            const float* const bs = lds[t & 1][1];
#pragma unroll
            for (int q = 0; q < TK / 16; ++q) {
                float4 a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[i] = *reinterpret_cast<const float4*>(as + tile_off(wm0 + i * 16 + l16, q * 4 + lq));
                    b[i] = *reinterpret_cast<const float4*>(bs + tile_off(wn0 + i * 16 + l16, q * 4 + lq));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(get(b[j], e), get(a[i], e), acc[i][j]);
            }
            if (t + 1 < steps) stage(t + 1, next);     // that buffer was read last in step t - 1, before its barrier
            __syncthreads();
        };
        float4 va[4], vb[4];
        if (steps > 0) { fetch(0, va); stage(0, va); }
        if (steps > 1) fetch(1, vb);
        __syncthreads();
        for (int t = 0; t < steps; t += 2) {
            body(t, vb, va);
            if (t + 1 < steps) body(t + 1, va, vb);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + wm0 + i * 16 + l16;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn0 + j * 16 + lq * 4;
            float* c = p.c + (int64_t)m * p.ldc + n;
            if (n < N)                                 // N and ldc are multiples of four
                *reinterpret_cast<float4*>(c) = make_float4(p.alpha * acc[i][j][0], p.alpha * acc[i][j][1],
                                                            p.alpha * acc[i][j][2], p.alpha * acc[i][j][3]);
        }
    }
}

int64_t tiles(const SgemmArgs& a, int ts) { return a.M <= 0 || a.N <= 0 ? 0 : (int64_t)((a.N + ts - 1) / ts) * ((a.M + ts - 1) / ts); }

// 64 x 64 tiles once they fill half the chip; below, the split kernel
bool use_tile(const SgemmArgs& a) { return tiles(a, 64) >= 128; }

int longest_k(const SgemmArgs& a) { return a.nseg > 1 && a.seg[1].K > a.seg[0].K ? a.seg[1].K : a.seg[0].K; }

template <bool A_KC, bool B_KC>
hipError_t launch_layout(const SgemmArgs& a, const SgemmArgs* b, hipStream_t st)
{
    if (!b && use_tile(a)) {
        sgemm_tile_kernel<A_KC, B_KC><<<dim3((unsigned)tiles(a, 64)), dim3(256), 0, st>>>(a);
        return hipGetLastError();
    }
    SgemmPair grp;
    grp.g[0] = a;
    grp.g[1] = b ? *b : a;
    grp.count0 = (int)tiles(a, 32);
    const dim3 grid((unsigned)(grp.count0 + (b ? tiles(*b, 32) : 0)));
    const int K = b && longest_k(*b) > longest_k(a) ? longest_k(*b) : longest_k(a);
    // sixteen waves where each still has a group of 16 k, four for the products over the rank
    if (K >= 256) sgemm_split_kernel<16, A_KC, B_KC><<<grid, dim3(64 * 16), 0, st>>>(grp);
    else sgemm_split_kernel<4, A_KC, B_KC><<<grid, dim3(64 * 4), 0, st>>>(grp);
    return hipGetLastError();
}

hipError_t dispatch(const SgemmArgs& a, const SgemmArgs* b, hipStream_t st)
{
    if (a.a_kcontig && a.b_kcontig) return launch_layout<true, true>(a, b, st);
    if (a.a_kcontig) return launch_layout<true, false>(a, b, st);
    if (!a.b_kcontig) return launch_layout<false, false>(a, b, st);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_sgemm_f32(const SgemmArgs& a, int trace_id, hipStream_t stream)
{
    if (a.M == 0 || a.N == 0) return hipSuccess;
    TraceScope ts(trace_id, stream);
    return dispatch(a, nullptr, stream);
}

bool sgemm_f32_pairs(const SgemmArgs& a, const SgemmArgs& b)
{
    return a.a_kcontig == b.a_kcontig && a.b_kcontig == b.b_kcontig && !use_tile(a) && !use_tile(b) && tiles(a, 32) > 0 &&
           tiles(b, 32) > 0;
}

hipError_t launch_sgemm_f32_pair(const SgemmArgs& a, const SgemmArgs& b, int trace_id, hipStream_t stream)
{
    TraceScope ts(trace_id, stream);
    return dispatch(a, &b, stream);
}

}  // namespace dora
