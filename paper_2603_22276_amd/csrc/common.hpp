// Shared declarations of the HIP translation units of libdora (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/dora.h"
#include "../../include/dora_measure.h"

namespace dora {

typedef uint16_t bf16_t;  // storage only; arithmetic is fp32

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ---- bf16 <-> fp32 on the device ------------------------------------------------------------
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// round-to-nearest-even, NaN kept quiet
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    return (f != f) ? 0x7fc0u : r;
}
// two fp32 -> packed bf16 pair with the hardware converter (v_cvt_pk_bf16_f32: nearest-even)
typedef __bf16 bf16x2_hw_t __attribute__((ext_vector_type(2)));
typedef float f32x2_hw_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    f32x2_hw_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_hw_t));
}

// ---- the two 16-bit storage types --------------------------------------------------------------
// Kernels that serve both take a DT template parameter; everything element-specific goes through
// Elem16<DT>: widening a packed pair, packing two fp32 with one rounding (nearest-even; fp16 overflows
// to infinity), and the matching MFMA.
enum { DT_BF16 = 0, DT_F16 = 1 };
struct f16_t { uint16_t bits; };  // distinct C++ type for fp16 storage (bf16_t is a plain uint16_t)
typedef _Float16 f16x2_hw_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

template <int DT> struct Elem16;
template <> struct Elem16<DT_BF16> {
    static __device__ __forceinline__ float lo(uint32_t packed) { return bf16_lo(packed); }
    static __device__ __forceinline__ float hi(uint32_t packed) { return bf16_hi(packed); }
    static __device__ __forceinline__ uint32_t pack2(float a, float b) { return pack_bf16x2(a, b); }
    static __device__ __forceinline__ f32x16_t mfma(bf16x8_t a, bf16x8_t b, f32x16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Elem16<DT_F16> {
    static __device__ __forceinline__ float lo(uint32_t packed)
    {
        return (float)__builtin_bit_cast(f16x2_hw_t, packed)[0];
    }
    static __device__ __forceinline__ float hi(uint32_t packed)
    {
        return (float)__builtin_bit_cast(f16x2_hw_t, packed)[1];
    }
    static __device__ __forceinline__ uint32_t pack2(float a, float b)
    {
        f32x2_hw_t v = {a, b};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_hw_t));
    }
    static __device__ __forceinline__ f32x16_t mfma(bf16x8_t a, bf16x8_t b, f32x16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0,
                                                      0);
    }
    static __device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0,
                                                      0);
    }
};

// Eq. 5 from its three fp32 terms: the sum in double, one rounding of the radicand and one of the root.  Clamps what is below
// zero; NaN is not, and propagates (App. C item 3).
__device__ __forceinline__ float radicand(float base_sq, float cross, float ba_sq, float two_s, float s2)
{
    const float rad = (float)((double)base_sq + (double)two_s * cross + (double)s2 * ba_sq);
    return (rad < 0.f) ? 0.f : rad;
}

// ---- kernel timing hook (see dora_trace_* in dora_measure.h) ------------------------------------------
void trace_begin(int kernel_id, hipStream_t stream);
void trace_end(int kernel_id, hipStream_t stream);

struct TraceScope {
    int id;
    hipStream_t st;
    TraceScope(int kernel_id, hipStream_t stream) : id(kernel_id), st(stream) { trace_begin(id, st); }
    ~TraceScope() { trace_end(id, st); }
};

// ---- bf16 MFMA GEMM family ---------------------------------------------------------------------
// C[M,N] = alpha * sum over segments of  Aop[m,k] * Bop[n,k]
// An operand is either K-contiguous (row-major [rows, K], ld = row stride) or K-strided
// (row-major [K, rows], ld = stride between consecutive k).
enum GemmEpilogue {
    EPI_STORE_BF16 = 0,  // C bf16 [M, ldc]
    EPI_STORE_F32 = 1,   // C fp32 [M, ldc]; with ksplit > 1 slice z goes to C + z*M*ldc
    EPI_ROWDOT = 2,      // no C; partial[z*tiles_n + tn][m] = sum_n acc[m,n] * R[m,n]  (+ base_sq of Aop rows)
    EPI_COMPOSE = 3      // C bf16 = colscale[n] * acc; optionally C2 bf16 = acc (the compose folded into the epilogue)
};

struct GemmSeg {
    const bf16_t* a;
    const bf16_t* b;
    int64_t lda, ldb;
    int K;
};

struct GemmArgs {
    GemmSeg seg[2];
    int nseg;
    int M, N;
    int a_kcontig, b_kcontig;  // layout of the M-side / N-side operand (both segments)
    int epilogue;
    float alpha;
    void* c;
    int64_t ldc;
    int ksplit;                // split of segment 0's K range (fp32 stores and row-dots only)
    int tag;                   // 0 or 1: selects a differently named (otherwise identical) kernel instance
    int dt;                    // DT_BF16 or DT_F16: element type of both operands, of a 16-bit C and of rowdot / colbias
    const float* colscale;     // EPI_COMPOSE: [N] fp32
    const bf16_t* colbias;     // EPI_COMPOSE: [N] bf16 added to the scaled output, or nullptr
    void* c2;                  // second output [M, ldc] bf16 or nullptr: the unscaled accumulator (compose epilogue),
                               // alpha2 * accumulator (bf16 store epilogue)
    float alpha2;
    // EPI_ROWDOT only
    const bf16_t* rowdot;      // R [M, ld_rowdot] bf16
    int64_t ld_rowdot;
    float* rowdot_partial;     // [ksplit * tiles_n][M]
    float* base_sq_partial;    // [ksplit][M] or nullptr
};

struct GemmPair {
    GemmArgs g[2];
    int count0;  // workgroups of g[0]; the rest of the grid belongs to g[1]
};

hipError_t launch_gemm_bf16(const GemmArgs& a, int trace_id, hipStream_t stream);
// two independent problems of the same kind (layouts, epilogue) in one launch; gemm_bf16_pairs: whether that is the cheaper way
// (their tiles share rounds of workgroups, and a launch is saved)
bool gemm_bf16_pairs(const GemmArgs& a, const GemmArgs& b);
hipError_t launch_gemm_bf16_pair(const GemmArgs& a, const GemmArgs& b, int trace_id, hipStream_t stream);
// n input gradients and m weight gradients (one or two of each) in one launch; gemm_bf16_grads_together: whether that is the
// cheaper way, and the only case that is taken
bool gemm_bf16_grads_together(const GemmArgs* dx, int n, const GemmArgs* w, int m);
hipError_t launch_gemm_bf16_grads(const GemmArgs* dx, int n, const GemmArgs* w, int m, int trace_id, hipStream_t stream);

// ---- forward of a few tokens (16-bit storage) ----------------------------------------------------
constexpr int64_t FEW_TOKENS_MAX = 64;
struct FewTokensArgs {
    const bf16_t* x;        // [T, K]
    const bf16_t* w;        // [N, K]: A for the h launch, W for the y launch
    int T, N, K, ksplit;
    float* part;            // h launch: [ksplit][T][N] fp32
    // y launch
    const float* h_part;    // [h_slices][T][r]
    int h_slices, r;
    const bf16_t* b;        // [N, r]
    float s, eps;
    const float *m, *c;     // [N]
    const bf16_t* bias;     // [N] or nullptr
    bf16_t *y, *inner, *h_out;   // [T, N]; [T, N] or nullptr; [T, r] or nullptr
};
int few_tokens_h_slices(int64_t tokens, int64_t r, int64_t d_in);
hipError_t launch_few_tokens_h(const FewTokensArgs& a, int dt, hipStream_t st);
hipError_t launch_few_tokens_y(const FewTokensArgs& a, int dt, hipStream_t st);

// ---- the three sums of the row norm (16-bit storage, norm_rows.hip) ------------------------------
constexpr int64_t NORM_ROWS_MAX_RANK = 384;
struct NormRowsArgs {
    const bf16_t* w;        // [d_out, d_in]
    const bf16_t* a;        // [r, d_in]
    const bf16_t* b;        // [d_out, r]
    int d_out, d_in, r;
    int slices, tiles_per_slice;   // slices of tiles_per_slice column tiles of 128 each; none of them empty
    float* part;            // [3][slices][d_out]: base_sq, cross, ba_sq
};
hipError_t launch_norm_rows(const NormRowsArgs& a, int dt, hipStream_t st);

// ---- fp32 products (sgemm_f32.hip) ----------------------------------------------------------------
// C[M,N] = alpha * rowscale[m] * sum over segments of  ascale[k] Aop[m,k] * Bop[n,k], operands K-contiguous or K-strided as in
// GemmArgs
struct RowScale {            // g as it is (m == nullptr), or formed from the row norm: m / max(g, eps), Eq. 6
    const float* g;          // nullptr: no scale
    const float* m;
    float eps;
};
struct SgemmSeg {
    const float* a;
    const float* b;
    int64_t lda, ldb;
    int K;
    bool scaled;             // ascale applies (M side K-contiguous, N side K-strided; in tiles only a scale that needs no forming)
};
struct SgemmArgs {
    SgemmSeg seg[2];
    int nseg;
    int M, N;
    int a_kcontig, b_kcontig;
    float alpha;
    float* c;
    int64_t ldc;
    RowScale ascale, rowscale;
    // composed != 0: the product is lora and c holds base; it receives y = base + (gm1 base + g (s lora)) (+ bias), inner
    // (may be nullptr) s lora + base
    int composed;
    const float *g, *gm1, *bias;
    float s;
    float* inner;
};
// the two stages of dm's column sum: partial[slab][j] = sum of dy[t][j] inner[t][j] over COLUMN_SUM_ROWS tokens; dm[j] = the
// sum of those in order / max(c[j], eps)
constexpr int COLUMN_SUM_ROWS = 64;
struct ColumnSum {
    const float *dy, *inner;
    int64_t tokens;
    int d_out;
    float* partial;
};
struct ColumnFinal {
    const float* partial;
    int slabs;
    const float* c;
    float eps;
    float* dm;
    int d_out;
};
struct ScaleOut {            // out[j] = the scale, j < n
    RowScale scale;
    float* out;
    int n;
};
inline int column_sum_slabs(int64_t tokens) { return (int)((tokens + COLUMN_SUM_ROWS - 1) / COLUMN_SUM_ROWS); }
// whether the product goes to tiles, where ascale has to be there as it is (m == nullptr)
bool f32_tiled(const SgemmArgs& a);
// up to three products and smaller pieces of work that do not need one another, in one launch
hipError_t launch_f32(const SgemmArgs* g, int n, const ColumnSum* sum, const ColumnFinal* fin, const ScaleOut* scale, int trace_id,
                      hipStream_t stream);
// norm of W + s B A from tiles of B A that stay in registers, Eq. 5 and (m != nullptr) Eq. 6 in the one launch; base_in: the
// base term, or nullptr; terms: [3, d_out] or nullptr; c may be nullptr where terms is not.  slices > 1: only the partial sums,
// to part [3][slices][d_out]
struct NormF32Args {
    const float *w, *a, *b;
    int d_out, d_in, r;
    const float* base_in;
    float two_s, s2;
    float *c, *terms;
    const float* m;
    float eps;
    float *g, *gm1;
    int slices;
    float* part;
    int row_blocks;         // of 16 rows to a workgroup: 1 or 2
};
hipError_t launch_norm_f32(const NormF32Args& a, hipStream_t stream);

// ---- element-wise / reduction kernels -----------------------------------------------------------
hipError_t launch_mag_scale(const float* m, const float* c, float eps, float* g, float* gm1, int d_out, hipStream_t st);
// write_delta: 0 out = base + delta (+ bias), 1 out = delta, 2 out += delta (+ bias)
hipError_t launch_compose_fwd(int dtype, const void* base, const void* lora, const float* g, const float* gm1,
                              const void* bias, float s, void* out, int write_delta, void* inner, int64_t tokens,
                              int d_out, hipStream_t st);
int compose_bwd_slabs(int64_t tokens, int d_out, int dtype);
// dzb != nullptr: also dzb = gm1 (.) dy (then gm1 must be given); m != nullptr: g is the row norm, and g and gm1 are
// formed from it, m and eps in the same launch
hipError_t launch_compose_bwd(int dtype, const void* dy, const void* inner, const float* g, const float* gm1, void* dz,
                              void* dzb, float* partial /* [slabs][d_out] or nullptr */, int64_t tokens, int d_out,
                              hipStream_t st, const float* m = nullptr, float eps = 0.f);
struct DmFinalArgs {          // dm[j] = sum of the slabs' partials / max(c[j], eps)
    const float* partial;
    int slabs;
    const float* c;
    float eps;
    float* dm;
    int d_out;
};
hipError_t launch_dm_final(const DmFinalArgs& a, hipStream_t st);
// G = sum of partials; Ghi + Glo ~ G as two 16-bit terms of element type dt (both may be nullptr)
hipError_t launch_gram_reduce(const float* partials, int ksplit, int r, float* G, bf16_t* Ghi, bf16_t* Glo, int dt,
                              hipStream_t st);
// Eq. 5 from partial sums.  c and / or terms ([3, d_out]: the summed base_sq, cross, ba_sq) may be nullptr
// m != nullptr: Eq. 6 in the same launch (g and / or gm1 from m, the norm just formed and eps)
struct NormFinalArgs {
    const float* base_p; int n_base;
    const float* cross_p; int n_cross;
    const float* ba_p; int n_ba;
    float two_s, s2;          // formed in double and rounded once (App. C item 3)
    float *c, *terms;
    int d_out;
    const float* m;
    float eps;
    float *g, *gm1;
};
inline NormFinalArgs norm_final_args(const float* base_p, int n_base, const float* cross_p, int n_cross, const float* ba_p, int n_ba,
                                     double s, float* c, float* terms, int d_out, const float* m = nullptr, float eps = 0.f,
                                     float* g = nullptr, float* gm1 = nullptr)
{
    return NormFinalArgs{base_p, n_base, cross_p, n_cross, ba_p, n_ba, (float)(2.0 * s), (float)(s * s), c, terms, d_out, m, eps, g, gm1};
}
hipError_t launch_norm_final(const NormFinalArgs& a, hipStream_t st);
// Small launches that nothing waits for yet: they ride in the next reduce launch of a split product, or are launched by
// launch_waiting where none came.
struct Waiting {
    bool norm = false, dm = false;
    NormFinalArgs norm_args;
    DmFinalArgs dm_args;
};
hipError_t launch_waiting(Waiting& w, hipStream_t st);
hipError_t launch_rownorm_s0_16(const bf16_t* W, int dt, float* c, int d_out, int d_in, bool squared, hipStream_t st);
// fp32: the row norms of W alone (or their squares); terms ([3, d_out]: base_sq, 0, 0) and c may be nullptr
hipError_t launch_rownorm_f32(const float* W, float* c, float* terms, int d_out, int d_in, bool squared, hipStream_t st);

// out[i] = sum over z (in order) of partials[z * n + i], written in the 16-bit storage dtype; out2 (may be nullptr)
// receives alpha2 times the same sum.  n a multiple of 8.  colscale != nullptr: rows of `cols` elements, out is
// colscale[col] times the sum (+ colbias[col] where given).
hipError_t launch_splitk_reduce(const float* partials, int ksplit, int64_t n, int dtype, void* out, float alpha2, void* out2,
                                hipStream_t st, const float* colscale = nullptr, const void* colbias = nullptr, int cols = 0,
                                Waiting* waiting = nullptr);

hipError_t launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t st);
hipError_t launch_mfma_probe(const void* operands, float* sink, int iters, int workgroups, hipStream_t st);

}  // namespace dora
