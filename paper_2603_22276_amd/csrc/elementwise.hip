// Element-wise and reduction kernels of the DoRA hot path: magnitude scale (Eq. 6), norm assembly
// (Eq. 5), compose forward (Sec. 3.1, App. C item 1), compose backward with the fused two-stage
// column reduction for the magnitude gradient (Sec. 3.2; Sec. 7 "LLM-guided optimization").
//
// All of these are HBM streams: every thread moves 16-byte vectors, a workgroup owns a fixed set
// of columns (so g / gm1 live in registers) and walks down a slab of token rows.
#include "common.hpp"

namespace dora {

namespace {

// Block shape of the compose passes: CW threads along the column direction (one 16-byte vector each), CH along
// the row direction, CW * CH = 256.  Measured inside the forward + backward sequence at 8192 x 8192: the forward
// pass (two tensors updated in place) is fastest with one thread row spanning 4 KB of every row it touches
// (256 x 1: 85 us against 95 us for 64 x 4); the backward pass (three separate streams) with 64 x 4 and short
// slabs (70 us against 83 / 95 us for 128 x 2 / 256 x 1).  The two passes are not independent: what the forward
// pass leaves behind in the memory system moves the backward pass by several microseconds, so they were tuned
// together, inside the sequence.
constexpr int BWD_CW = 64, BWD_CH = 4;

// 16-byte store with the non-temporal hint, for outputs nothing reads soon; on this part the hint lifts a
// 2-read/2-write stream from ~5.4 to ~6.9 TB/s in isolation.
typedef unsigned int u32x4_nt_t __attribute__((ext_vector_type(4)));
template <typename R>
__device__ __forceinline__ void store_plain(void* p, const R& v)
{
    *reinterpret_cast<R*>(p) = v;
}
template <typename R>
__device__ __forceinline__ void store_stream(void* p, const R& v)
{
    static_assert(sizeof(R) == 16, "16-byte vectors only");
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4_nt_t, v), reinterpret_cast<u32x4_nt_t*>(p));
}

template <typename T> struct Vec;
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    typedef uint4 raw_t;
    static __device__ __forceinline__ void unpack(const raw_t& r, float* f)
    {
        f[0] = bf16_lo(r.x); f[1] = bf16_hi(r.x); f[2] = bf16_lo(r.y); f[3] = bf16_hi(r.y);
        f[4] = bf16_lo(r.z); f[5] = bf16_hi(r.z); f[6] = bf16_lo(r.w); f[7] = bf16_hi(r.w);
    }
    static __device__ __forceinline__ raw_t pack(const float* f)
    {
        raw_t r;
        r.x = pack_bf16x2(f[0], f[1]); r.y = pack_bf16x2(f[2], f[3]);
        r.z = pack_bf16x2(f[4], f[5]); r.w = pack_bf16x2(f[6], f[7]);
        return r;
    }
};
template <> struct Vec<f16_t> {
    static constexpr int N = 8;
    typedef uint4 raw_t;
    typedef Elem16<DT_F16> E;
    static __device__ __forceinline__ void unpack(const raw_t& r, float* f)
    {
        f[0] = E::lo(r.x); f[1] = E::hi(r.x); f[2] = E::lo(r.y); f[3] = E::hi(r.y);
        f[4] = E::lo(r.z); f[5] = E::hi(r.z); f[6] = E::lo(r.w); f[7] = E::hi(r.w);
    }
    static __device__ __forceinline__ raw_t pack(const float* f)
    {
        raw_t r;
        r.x = E::pack2(f[0], f[1]); r.y = E::pack2(f[2], f[3]);
        r.z = E::pack2(f[4], f[5]); r.w = E::pack2(f[6], f[7]);
        return r;
    }
};
template <> struct Vec<float> {
    static constexpr int N = 4;
    typedef float4 raw_t;
    static __device__ __forceinline__ void unpack(const raw_t& r, float* f) { f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w; }
    static __device__ __forceinline__ raw_t pack(const float* f) { return make_float4(f[0], f[1], f[2], f[3]); }
};

// p[0] + p[stride] + ... in index order, U loads in flight: the launches that sum a handful of partials per thread are
// bound by the latency of their loads, one after the other when each waits for the sum so far (U = 1).  A norm over weight
// sets of 1.2 GB in turn, one load at a time -> this: 8192 x 8192, r 128 60.1 -> 53.8 us; 4096 x 4096, r 384 47.5 -> 43.1;
// 1024 x 4096, r 64 30.5 -> 24.1.
template <int U>
__device__ __forceinline__ float sum_partials(const float* __restrict__ p, int n, int64_t stride)
{
    float acc = 0.f;
    for (int i = 0; i < n; i += U) {
        float v[U];
#pragma unroll
        for (int e = 0; e < U; ++e) v[e] = p[(int64_t)(i + e < n ? i + e : n - 1) * stride];
#pragma unroll
        for (int e = 0; e < U; ++e) acc += i + e < n ? v[e] : 0.f;
    }
    return acc;
}

// ------------------------------------------------------------------------------------------------
// Eq. 6 and the explicit small correction of Sec. 3.1.
__global__ void mag_scale_kernel(const float* __restrict__ m, const float* __restrict__ c, float eps,
                                 float* __restrict__ g, float* __restrict__ gm1, int d_out)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= d_out) return;
    float cj = c[j];
    float cc = (cj < eps) ? eps : cj;  // NaN stays NaN
    float mj = m[j];
    if (g) g[j] = mj / cc;
    if (gm1) gm1[j] = (mj - cc) / cc;  // the subtraction is exact when m/cc is within [1/2, 2]
}

// Eq. 5 from the partial sums the norm kernels left behind, in a fixed order: NF_H threads per row take every NF_H-th each.
// terms != nullptr: the three summed terms are also written, as rows of a [3, d_out] array (base_sq,
// cross, ba_sq); c == nullptr: only the terms are wanted.  m != nullptr: Eq. 6 follows in the same launch
// (g and / or gm1, exactly as mag_scale_kernel forms them).
constexpr int NF_W = 32, NF_H = 8;
__device__ __forceinline__ void norm_final(const NormFinalArgs& p, int block)
{
    __shared__ float red[3][NF_H][NF_W];
    const int d_out = p.d_out, x = threadIdx.x % NF_W, y = threadIdx.x / NF_W, j = block * NF_W + x;
    const int64_t first = (int64_t)y * d_out + j, stride = (int64_t)NF_H * d_out;
    auto share = [&](int n) { return n > y ? (n - y + NF_H - 1) / NF_H : 0; };
    if (j < d_out) {
        red[0][y][x] = sum_partials<4>(p.base_p + first, share(p.n_base), stride);
        red[1][y][x] = sum_partials<4>(p.cross_p + first, share(p.n_cross), stride);
        red[2][y][x] = sum_partials<4>(p.ba_p + first, share(p.n_ba), stride);
    }
    __syncthreads();
    if (y != 0 || j >= d_out) return;
    // (in double: eight sums of a like size one after the other in fp32 cost the norm 1e-8 to 2e-8 of its 5e-8)
    float sum[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double v = red[k][0][x];
#pragma unroll
        for (int i = 1; i < NF_H; ++i) v += red[k][i][x];
        sum[k] = (float)v;
    }
    const float base_sq = sum[0], cross = sum[1], ba = sum[2];
    if (p.terms) {
        p.terms[j] = base_sq;
        p.terms[(int64_t)d_out + j] = cross;
        p.terms[2 * (int64_t)d_out + j] = ba;
    }
    if (!p.c) return;
    const float cj = __fsqrt_rn(radicand(base_sq, cross, ba, p.two_s, p.s2));
    p.c[j] = cj;
    if (p.m) {
        float cc = (cj < p.eps) ? p.eps : cj;
        float mj = p.m[j];
        if (p.g) p.g[j] = mj / cc;
        if (p.gm1) p.gm1[j] = (mj - cc) / cc;
    }
}
__global__ __launch_bounds__(NF_W* NF_H) void norm_final_kernel(NormFinalArgs p) { norm_final(p, blockIdx.x); }

// G = sum of split-K partials (fixed order), and its two-term 16-bit expansion G ~ Ghi + Glo.
template <int DT>
__global__ void gram_reduce_kernel(const float* __restrict__ p, int ksplit, int rr, float* __restrict__ G,
                                   bf16_t* __restrict__ Ghi, bf16_t* __restrict__ Glo)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rr) return;
    const float acc = sum_partials<16>(p + i, ksplit, rr);
    if (G) G[i] = acc;
    if (!Ghi) return;
    typedef Elem16<DT> E;
    uint32_t hi = E::pack2(acc, 0.f) & 0xffffu;
    float rem = acc - E::lo(hi);     // exact: the leading bits of acc cancel
    Ghi[i] = (bf16_t)hi;
    Glo[i] = (bf16_t)(E::pack2(rem, 0.f) & 0xffffu);
}

// Second stage of dm's column sum: dm[j] = (sum over slabs, in slab order) / max(c[j], eps).  32 columns per workgroup, H threads
// per column; the slabs go in 32 contiguous ranges whose sums are added in order, 32 / H of them to a thread, so that dm does not
// depend on which launch forms it.
constexpr int DMF_W = 32, DMF_RANGES = 32;
template <int H>
__device__ __forceinline__ void dm_final(const DmFinalArgs& p, int block)
{
    constexpr int PER = DMF_RANGES / H, U = PER == 1 ? 8 : 4;      // loads of a range in flight
    __shared__ float red[DMF_RANGES][DMF_W];
    const int x = threadIdx.x % DMF_W, y = threadIdx.x / DMF_W, j = block * DMF_W + x;
    const int length = (p.slabs + DMF_RANGES - 1) / DMF_RANGES;
    float acc[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) acc[q] = 0.f;
    if (j < p.d_out)
        for (int k = 0; k < length; k += U) {
            float v[PER][U];
#pragma unroll
            for (int q = 0; q < PER; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int z = (y * PER + q) * length + k + u;
                    v[q][u] = p.partial[(int64_t)(z < p.slabs ? z : p.slabs - 1) * p.d_out + j];
                }
#pragma unroll
            for (int q = 0; q < PER; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u) acc[q] += k + u < length && (y * PER + q) * length + k + u < p.slabs ? v[q][u] : 0.f;
        }
#pragma unroll
    for (int q = 0; q < PER; ++q) red[y * PER + q][x] = acc[q];
    __syncthreads();
    if (y == 0 && j < p.d_out) {
        float v = red[0][x];
        for (int i = 1; i < DMF_RANGES; ++i) v += red[i][x];
        const float cj = p.c[j];
        p.dm[j] = v / ((cj < p.eps) ? p.eps : cj);
    }
}
__global__ __launch_bounds__(DMF_W * 32) void dm_final_kernel(DmFinalArgs p) { dm_final<32>(p, blockIdx.x); }

struct Riders {
    NormFinalArgs norm;
    DmFinalArgs dm;
    int norm_blocks, dm_blocks;
};

// Sum of the K slices of a split contraction, in slice order, rounded once to the storage dtype; with colscale the
// first output is y = g (.) inner (+ bias), formed from the fp32 sum.
// Its first workgroups do what other small work is due, Eq. 5 and 6 or dm's second stage, of a handful of partials per column:
// launches of their own take 2.7 to 5 us each, nearly all of it the launch.  (1024 x 4096, r 64, 512 tokens, forward and backward
// 74.9 -> 70.3 us; 4096 x 4096, 4096 tokens, forward 160.2 -> 157.6; 2056 x 3000, 1501 tokens with dropout 195.9 -> 191.9.)
template <typename T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ p, int ksplit, int64_t n, T* __restrict__ out,
                                     float alpha2, T* __restrict__ out2, const float* __restrict__ colscale,
                                     const T* __restrict__ colbias, int cols, Riders riders)
{
    typedef Vec<T> V;
    constexpr int N = V::N;
    int block = blockIdx.x;
    if (block < riders.norm_blocks) return norm_final(riders.norm, block);
    block -= riders.norm_blocks;
    if (block < riders.dm_blocks) return dm_final<8>(riders.dm, block);
    block -= riders.dm_blocks;
    const int64_t i = ((int64_t)block * blockDim.x + threadIdx.x) * N;
    if (i >= n) return;
    float acc[N];
#pragma unroll
    for (int e = 0; e < N; ++e) acc[e] = 0.f;
    constexpr int U = 4;                               // slices in flight
    for (int z = 0; z < ksplit; z += U) {
        float4 v[U][N / 4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < N / 4; ++e)
                v[u][e] = *reinterpret_cast<const float4*>(p + (int64_t)(z + u < ksplit ? z + u : ksplit - 1) * n + i + e * 4);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (z + u < ksplit)
#pragma unroll
                for (int e = 0; e < N / 4; ++e) {
                    acc[4 * e] += v[u][e].x; acc[4 * e + 1] += v[u][e].y; acc[4 * e + 2] += v[u][e].z; acc[4 * e + 3] += v[u][e].w;
                }
    }
    if (colscale) {
        const int col = (int)(i % cols);
        float v[N], bv[N];
#pragma unroll
        for (int e = 0; e < N; ++e) bv[e] = 0.f;
        if (colbias) V::unpack(*reinterpret_cast<const typename V::raw_t*>(colbias + col), bv);
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = fmaf(colscale[col + e], acc[e], bv[e]);
        *reinterpret_cast<typename V::raw_t*>(out + i) = V::pack(v);
    } else {
        *reinterpret_cast<typename V::raw_t*>(out + i) = V::pack(acc);
    }
    if (out2) {
#pragma unroll
        for (int e = 0; e < N; ++e) acc[e] *= alpha2;
        *reinterpret_cast<typename V::raw_t*>(out2 + i) = V::pack(acc);
    }
}

// fp32, W alone (s == 0, Algorithm 1, notes; the cached base term of Sec. 2.3): one row per wavefront.  squared: write the
// sum itself, not its root.  terms != nullptr: base_sq, and zeros for cross and ba_sq.
__global__ void rownorm_f32_kernel(const float* __restrict__ W, float* __restrict__ c, float* __restrict__ terms, int d_out, int d_in,
                                   bool squared)
{
    int lane = threadIdx.x & 63;
    int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= d_out) return;
    float base_sq = 0.f;
    const float* w = W + (int64_t)row * d_in;
    for (int k = lane; k < d_in; k += 64) { float v = w[k]; base_sq = fmaf(v, v, base_sq); }
    for (int o = 32; o > 0; o >>= 1) base_sq += __shfl_xor(base_sq, o);
    if (lane == 0) {
        if (terms) {
            terms[row] = base_sq;
            terms[(int64_t)d_out + row] = 0.f;
            terms[2 * (int64_t)d_out + row] = 0.f;
        }
        if (c) c[row] = squared ? base_sq : __fsqrt_rn(base_sq);
    }
}

// s == 0 (Algorithm 1, notes): the norm is the row norm of W alone.  One wavefront per row, 16-bit storage.
template <typename T>
__global__ void rownorm_s0_16_kernel(const T* __restrict__ W, float* __restrict__ c, int d_out, int d_in,
                                     bool squared)
{
    int lane = threadIdx.x & 63;
    int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= d_out) return;
    const T* w = W + (int64_t)row * d_in;
    float acc = 0.f;
    for (int k = lane * 8; k < d_in; k += 64 * 8) {
        uint4 v = *reinterpret_cast<const uint4*>(w + k);
        float f[8];
        Vec<T>::unpack(v, f);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fmaf(f[i], f[i], acc);
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) c[row] = squared ? acc : __fsqrt_rn(acc);
}

// ------------------------------------------------------------------------------------------------
// Compose forward.  delta = gm1*base + g*(s*lora);  out = delta or base + delta;  inner = s*lora + base.
// OUTMODE: 0 = no out tensor (inner only), 1 = out = base + delta, 2 = out = delta, 3 = out += delta (the
// frozen layer's output is already in out and base is the adapter branch's own base, App. B "Chunked
// dropout path").
template <typename T, int OUTMODE, bool INNER, int CW, int CH>
__global__ __launch_bounds__(CW* CH) void compose_fwd_kernel(const T* base_, const T* lora_,  // out may alias base, inner may alias lora
                                                             
                                                              const float* __restrict__ g, const float* __restrict__ gm1,
                                                              const T* __restrict__ bias,  // added to out = base + delta only; may be null
                                                              float s, T* out_, T* inner_, int64_t tokens, int d_out,
                                                              int rows_per_wg, int col_blocks)
{
    typedef Vec<T> V;
    typedef typename V::raw_t raw_t;
    constexpr int N = V::N;
    // one-dimensional grid (no 65535 limit on either extent): consecutive workgroups take neighbouring
    // column blocks of one row slab
    const int col_block = blockIdx.x % col_blocks;
    const int64_t slab = blockIdx.x / col_blocks;
    const int col = (col_block * CW + threadIdx.x) * N;
    if (col >= d_out) return;
    float gv[N], g1[N], bv[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        gv[i] = g[col + i];
        g1[i] = gm1 ? gm1[col + i] : gv[i] - 1.0f;
        bv[i] = 0.f;
    }
    if ((OUTMODE == 1 || OUTMODE == 3) && bias) V::unpack(*reinterpret_cast<const raw_t*>(bias + col), bv);
    const int64_t row_begin = slab * rows_per_wg;
    int64_t row_end = row_begin + rows_per_wg;
    if (row_end > tokens) row_end = tokens;
    constexpr int UNROLL = 4;
    for (int64_t row = row_begin + threadIdx.y; row < row_end; row += CH * UNROLL) {
        raw_t b[UNROLL], l[UNROLL], y0[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int64_t rr = row + u * CH;
            if (rr < row_end) {
                b[u] = *reinterpret_cast<const raw_t*>(base_ + rr * d_out + col);
                l[u] = *reinterpret_cast<const raw_t*>(lora_ + rr * d_out + col);
                if (OUTMODE == 3) y0[u] = *reinterpret_cast<const raw_t*>(out_ + rr * d_out + col);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int64_t rr = row + u * CH;
            if (rr < row_end) {
                float bf[N], lf[N], of[N], inf[N], yf[N];
                V::unpack(b[u], bf);
                V::unpack(l[u], lf);
                if (OUTMODE == 3) V::unpack(y0[u], yf);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    float sl = s * lf[i];                        // canonical order: s*lora first, then g*(.)
                    float delta = fmaf(g1[i], bf[i], gv[i] * sl);
                    of[i] = (OUTMODE == 2) ? delta : (((OUTMODE == 3) ? yf[i] : bf[i]) + delta) + bv[i];
                    inf[i] = sl + bf[i];
                }
                // y leaves with the streaming hint; inner with a plain store, so that the pass that reads it next (the
                // compose backward of the same module, right away when inner was recomputed) can find it in cache
                if (OUTMODE != 0) store_stream(out_ + rr * d_out + col, V::pack(of));
                if (INNER) store_plain(inner_ + rr * d_out + col, V::pack(inf));
            }
        }
    }
}

// Compose backward: dz = g*dy, and (DM) the first stage of the column sum of dy*inner over this slab.
// SPLIT: also dzb = (g-1)*dy, the gradient reaching the adapter branch's own base when that branch has an
// input of its own (dz then reaches lora only, scaled by s in the products that follow).  m != nullptr: g is the row
// norm and Eq. 6 is formed here, as in mag_scale_kernel: a launch of d_out threads costs more than a few divisions per
// workgroup of a pass over [tokens, d_out].
template <typename T, bool DM, bool SPLIT, int CW, int CH>
__global__ __launch_bounds__(CW* CH) void compose_bwd_kernel(const T* __restrict__ dy_, const T* __restrict__ inner_,
                                                              const float* __restrict__ g, const float* __restrict__ gm1,
                                                              T* __restrict__ dz_, T* __restrict__ dzb_,
                                                              float* __restrict__ partial, int64_t tokens, int d_out,
                                                              int rows_per_wg, int col_blocks, const float* __restrict__ m,
                                                              float eps)
{
    typedef Vec<T> V;
    typedef typename V::raw_t raw_t;
    constexpr int N = V::N;
    __shared__ float red[CH][CW * N];
    const int col_block = blockIdx.x % col_blocks;
    const int64_t slab = blockIdx.x / col_blocks;
    const int col = (col_block * CW + threadIdx.x) * N;
    const bool active = col < d_out;
    float gv[N], g1[N], acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        gv[i] = active ? g[col + i] : 0.f;
        g1[i] = (SPLIT && active && !m) ? gm1[col + i] : 0.f;
        acc[i] = 0.f;
    }
    if (m && active) {   // g is the row norm
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float cc = (gv[i] < eps) ? eps : gv[i], mj = m[col + i];
            gv[i] = mj / cc;
            if (SPLIT) g1[i] = (mj - cc) / cc;
        }
    }
    const int64_t row_begin = slab * rows_per_wg;
    int64_t row_end = row_begin + rows_per_wg;
    if (row_end > tokens) row_end = tokens;
    constexpr int UNROLL = 4, STEP = CH * UNROLL;
    if (active) {
        // Two register sets used in turn (no copies between them): the loads of batch b+1 are in flight while
        // batch b is reduced and stored.  Batches that lie wholly inside the slab take loads and stores without
        // per-row conditions, so the waits the compiler places count exactly the loads still outstanding.
        raw_t da[UNROLL], ia[UNROLL], db[UNROLL], ib[UNROLL];
        auto load_full = [&](int64_t row, raw_t (&dd)[UNROLL], raw_t (&ii)[UNROLL]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int64_t rr = row + u * CH;
                dd[u] = *reinterpret_cast<const raw_t*>(dy_ + rr * d_out + col);
                if (DM) ii[u] = *reinterpret_cast<const raw_t*>(inner_ + rr * d_out + col);
            }
        };
        auto row_work = [&](int64_t rr, const raw_t& dv, const raw_t& iv) {
            float df[N], nf[N], zf[N], zb[N];
            V::unpack(dv, df);
            if (DM) V::unpack(iv, nf);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                zf[i] = gv[i] * df[i];
                if (SPLIT) zb[i] = g1[i] * df[i];
                if (DM) acc[i] = fmaf(df[i], nf[i], acc[i]);
            }
            store_stream(dz_ + rr * d_out + col, V::pack(zf));   // (a plain store here slows the dh product by 14 us)
            if (SPLIT) store_stream(dzb_ + rr * d_out + col, V::pack(zb));
        };
        auto work_full = [&](int64_t row, const raw_t (&dd)[UNROLL], const raw_t (&ii)[UNROLL]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) row_work(row + u * CH, dd[u], ii[u]);
        };
        const int nfull = (int)((row_end - row_begin) / STEP);   // uniform over the workgroup
        int64_t row = row_begin + threadIdx.y;
        if (nfull > 0) load_full(row, da, ia);
        for (int b = 0; b < nfull; b += 2) {
            if (b + 1 < nfull) load_full(row + STEP, db, ib);
            work_full(row, da, ia);
            row += STEP;
            if (b + 1 >= nfull) break;
            if (b + 2 < nfull) load_full(row + STEP, da, ia);
            work_full(row, db, ib);
            row += STEP;
        }
        // ragged end of the slab (fewer than STEP rows)
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int64_t rr = row + u * CH;
            if (rr < row_end) {
                raw_t dv = *reinterpret_cast<const raw_t*>(dy_ + rr * d_out + col), iv = dv;
                if (DM) iv = *reinterpret_cast<const raw_t*>(inner_ + rr * d_out + col);
                row_work(rr, dv, iv);
            }
        }
    }
    if (DM) {
#pragma unroll
        for (int i = 0; i < N; ++i) red[threadIdx.y][threadIdx.x * N + i] = acc[i];
        __syncthreads();
        if (threadIdx.y == 0 && active) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float v = red[0][threadIdx.x * N + i];
                for (int y = 1; y < CH; ++y) v += red[y][threadIdx.x * N + i];  // fixed order
                partial[slab * d_out + col + i] = v;
            }
        }
    }
}

}  // namespace

hipError_t launch_mag_scale(const float* m, const float* c, float eps, float* g, float* gm1, int d_out, hipStream_t st)
{
    if (d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_MAG_SCALE, st);
    mag_scale_kernel<<<dim3((d_out + 255) / 256), dim3(256), 0, st>>>(m, c, eps, g, gm1, d_out);
    return hipGetLastError();
}

hipError_t launch_norm_final(const NormFinalArgs& a, hipStream_t st)
{
    if (a.d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_NORM_FINAL, st);
    norm_final_kernel<<<dim3((a.d_out + NF_W - 1) / NF_W), dim3(NF_W * NF_H), 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_waiting(Waiting& w, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (w.norm) e = launch_norm_final(w.norm_args, st);
    if (e == hipSuccess && w.dm) e = launch_dm_final(w.dm_args, st);
    w.norm = w.dm = false;
    return e;
}

hipError_t launch_gram_reduce(const float* partials, int ksplit, int r, float* G, bf16_t* Ghi, bf16_t* Glo, int dt,
                              hipStream_t st)
{
    int rr = r * r;
    if (rr == 0) return hipSuccess;
    TraceScope ts(DORA_K_GRAM_REDUCE, st);
    if (dt == DT_F16) gram_reduce_kernel<DT_F16><<<dim3((rr + 255) / 256), dim3(256), 0, st>>>(partials, ksplit, rr, G, Ghi, Glo);
    else gram_reduce_kernel<DT_BF16><<<dim3((rr + 255) / 256), dim3(256), 0, st>>>(partials, ksplit, rr, G, Ghi, Glo);
    return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float* partials, int ksplit, int64_t n, int dtype, void* out, float alpha2, void* out2,
                                hipStream_t st, const float* colscale, const void* colbias, int cols, Waiting* waiting)
{
    if (n == 0) return waiting ? launch_waiting(*waiting, st) : hipSuccess;
    TraceScope ts(DORA_K_SPLITK_REDUCE, st);
    constexpr int per = 8;
    Riders r{};
    if (waiting && waiting->norm) { r.norm = waiting->norm_args; r.norm_blocks = (r.norm.d_out + NF_W - 1) / NF_W; }
    if (waiting && waiting->dm) { r.dm = waiting->dm_args; r.dm_blocks = (r.dm.d_out + DMF_W - 1) / DMF_W; }
    if (waiting) waiting->norm = waiting->dm = false;
    dim3 grid((unsigned)(r.norm_blocks + r.dm_blocks + (n / per + 255) / 256)), block(256);
    if (dtype == DORA_BF16)
        splitk_reduce_kernel<bf16_t><<<grid, block, 0, st>>>(partials, ksplit, n, (bf16_t*)out, alpha2, (bf16_t*)out2, colscale,
                                                    (const bf16_t*)colbias, cols, r);
    else
        splitk_reduce_kernel<f16_t><<<grid, block, 0, st>>>(partials, ksplit, n, (f16_t*)out, alpha2, (f16_t*)out2, colscale,
                                                    (const f16_t*)colbias, cols, r);
    return hipGetLastError();
}

hipError_t launch_rownorm_s0_16(const bf16_t* W, int dt, float* c, int d_out, int d_in, bool squared, hipStream_t st)
{
    if (d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_NORM_FINAL, st);
    if (dt == DT_F16)
        rownorm_s0_16_kernel<f16_t><<<dim3((d_out + 3) / 4), dim3(256), 0, st>>>((const f16_t*)W, c, d_out, d_in, squared);
    else
        rownorm_s0_16_kernel<bf16_t><<<dim3((d_out + 3) / 4), dim3(256), 0, st>>>(W, c, d_out, d_in, squared);
    return hipGetLastError();
}

hipError_t launch_rownorm_f32(const float* W, float* c, float* terms, int d_out, int d_in, bool squared, hipStream_t st)
{
    if (d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_NORM_FINAL, st);
    rownorm_f32_kernel<<<dim3((d_out + 3) / 4), dim3(256), 0, st>>>(W, c, terms, d_out, d_in, squared);
    return hipGetLastError();
}

// Rows per workgroup: 128 forward, 32 backward (measured inside the whole forward + backward sequence);
// shorter ones are chosen only when the launch would otherwise leave CUs without work.
static int slab_rows(int preferred, int64_t tokens, int d_out, int dtype, int CW)
{
    const int n = dtype == DORA_F32 ? 4 : 8;
    const int64_t col_blocks = (d_out / n + CW - 1) / CW;
    for (int rows = preferred; rows > 16; rows >>= 1)
        if (col_blocks * ((tokens + rows - 1) / rows) >= 512) return rows;
    return 16;
}

template <typename T>
static hipError_t compose_fwd_t(const void* base, const void* lora, const float* g, const float* gm1, const void* bias,
                                float s, void* out, int write_delta, void* inner, int64_t tokens, int d_out,
                                hipStream_t st)
{
    constexpr int N = Vec<T>::N;
    int cpr = d_out / N;
    // the widest block that leaves no thread without a column
    const int CW = cpr >= 256 ? 256 : (cpr >= 128 ? 128 : 64), CH = 256 / CW;
    const int FWD_ROWS_PER_WG = slab_rows(128, tokens, d_out, sizeof(T) == 2 ? DORA_BF16 : DORA_F32, CW);
    const int col_blocks = (cpr + CW - 1) / CW;
    dim3 grid((unsigned)(col_blocks * ((tokens + FWD_ROWS_PER_WG - 1) / FWD_ROWS_PER_WG)));
    dim3 block(CW, CH);
    const T* b = (const T*)base;
    const T* l = (const T*)lora;
    T* o = (T*)out;
    T* in = (T*)inner;
#define DORA_LAUNCH_FWD_S(D, I, W_, H_) \
    compose_fwd_kernel<T, D, I, W_, H_><<<grid, block, 0, st>>>(b, l, g, gm1, (const T*)bias, s, o, in, tokens, d_out, FWD_ROWS_PER_WG, col_blocks)
#define DORA_LAUNCH_FWD(D, I)                                        \
    do {                                                             \
        if (CW == 256) DORA_LAUNCH_FWD_S(D, I, 256, 1);              \
        else if (CW == 128) DORA_LAUNCH_FWD_S(D, I, 128, 2);         \
        else DORA_LAUNCH_FWD_S(D, I, 64, 4);                         \
    } while (0)
    if (!out) {
        if constexpr (sizeof(T) == 2) DORA_LAUNCH_FWD(0, true);
        else return hipErrorInvalidValue;              // fp32 forms inner alone in the launch of lora
    }
    else if (write_delta == 2) { if (inner) DORA_LAUNCH_FWD(3, true); else DORA_LAUNCH_FWD(3, false); }
    else if (write_delta) { if (inner) DORA_LAUNCH_FWD(2, true); else DORA_LAUNCH_FWD(2, false); }
    else { if (inner) DORA_LAUNCH_FWD(1, true); else DORA_LAUNCH_FWD(1, false); }
#undef DORA_LAUNCH_FWD
#undef DORA_LAUNCH_FWD_S
    return hipGetLastError();
}

hipError_t launch_compose_fwd(int dtype, const void* base, const void* lora, const float* g, const float* gm1,
                              const void* bias, float s, void* out, int write_delta, void* inner, int64_t tokens,
                              int d_out, hipStream_t st)
{
    if (tokens == 0 || d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_COMPOSE_FWD, st);
    if (dtype == DORA_BF16)
        return compose_fwd_t<bf16_t>(base, lora, g, gm1, bias, s, out, write_delta, inner, tokens, d_out, st);
    if (dtype == DORA_F16)
        return compose_fwd_t<f16_t>(base, lora, g, gm1, bias, s, out, write_delta, inner, tokens, d_out, st);
    return compose_fwd_t<float>(base, lora, g, gm1, bias, s, out, write_delta, inner, tokens, d_out, st);
}

static int compose_bwd_rows(int64_t tokens, int d_out, int dtype) { return slab_rows(32, tokens, d_out, dtype, BWD_CW); }

int compose_bwd_slabs(int64_t tokens, int d_out, int dtype)
{
    const int rows = compose_bwd_rows(tokens, d_out, dtype);
    return (int)((tokens + rows - 1) / rows);
}

template <typename T>
static hipError_t compose_bwd_t(const void* dy, const void* inner, const float* g, const float* gm1, void* dz, void* dzb,
                                float* partial, int64_t tokens, int d_out, hipStream_t st, const float* m, float eps)
{
    constexpr int N = Vec<T>::N;
    int cpr = d_out / N;
    const int dtype = sizeof(T) == 2 ? DORA_BF16 : DORA_F32;
    const int BWD_ROWS_PER_WG = compose_bwd_rows(tokens, d_out, dtype);
    const int col_blocks = (cpr + BWD_CW - 1) / BWD_CW;
    dim3 grid((unsigned)((int64_t)col_blocks * compose_bwd_slabs(tokens, d_out, dtype)));
    dim3 block(BWD_CW, BWD_CH);
#define DORA_LAUNCH_BWD(DM, SP)                                                                                   \
    compose_bwd_kernel<T, DM, SP, BWD_CW, BWD_CH><<<grid, block, 0, st>>>((const T*)dy, (const T*)inner, g, gm1, (T*)dz, (T*)dzb, partial, \
                                                           tokens, d_out, BWD_ROWS_PER_WG, col_blocks, m, eps)
    if (partial) { if (dzb) DORA_LAUNCH_BWD(true, true); else DORA_LAUNCH_BWD(true, false); }
    else { if (dzb) DORA_LAUNCH_BWD(false, true); else DORA_LAUNCH_BWD(false, false); }
#undef DORA_LAUNCH_BWD
    return hipGetLastError();
}

hipError_t launch_compose_bwd(int dtype, const void* dy, const void* inner, const float* g, const float* gm1, void* dz,
                              void* dzb, float* partial, int64_t tokens, int d_out, hipStream_t st, const float* m,
                              float eps)
{
    if (tokens == 0 || d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_COMPOSE_BWD, st);
    if (dtype == DORA_BF16) return compose_bwd_t<bf16_t>(dy, inner, g, gm1, dz, dzb, partial, tokens, d_out, st, m, eps);
    if (dtype == DORA_F16) return compose_bwd_t<f16_t>(dy, inner, g, gm1, dz, dzb, partial, tokens, d_out, st, m, eps);
    return compose_bwd_t<float>(dy, inner, g, gm1, dz, dzb, partial, tokens, d_out, st, m, eps);
}

hipError_t launch_dm_final(const DmFinalArgs& a, hipStream_t st)
{
    if (a.d_out == 0) return hipSuccess;
    TraceScope ts(DORA_K_DM_FINAL, st);
    dm_final_kernel<<<dim3((a.d_out + DMF_W - 1) / DMF_W), dim3(DMF_W * 32), 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace dora
