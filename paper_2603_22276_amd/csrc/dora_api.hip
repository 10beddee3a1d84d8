// C ABI of libdora: argument validation, workspace layout and the kernel sequence of each entry
// point.  Every step of the hot path runs in the kernels of this library; there is no fallback.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "common.hpp"

// Scratch of the entry point that allocates nothing (dora_norm_static): one file-scope device array,
// held by every GPU the library runs on until the process ends.  In host code the array's name is only
// a stand-in; the device address is looked up once per device and used from then on.
#define DORA_STATIC_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[DORA_STATIC_SCRATCH_BYTES];

namespace dora {

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES];  // per device: address of that device's copy of `scratch`

// Device address of the current device's scratch array (nullptr on failure).
void* static_scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

// ------------------------------------------------------------------------------------------------
// kernel timing (dora_trace_*)
namespace {
struct TraceRec { int id; hipEvent_t e0, e1; };
bool g_trace_on = false;
uint64_t g_trace_mask = ~0ull;
std::vector<TraceRec> g_trace_recs;          // launches since the last collect
std::vector<hipEvent_t> g_event_pool;        // recycled events
double g_trace_ms[DORA_K_COUNT];
int64_t g_trace_n[DORA_K_COUNT];
hipEvent_t g_pending_start = nullptr;

hipEvent_t get_event()
{
    if (!g_event_pool.empty()) { hipEvent_t e = g_event_pool.back(); g_event_pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}
}  // namespace

void trace_begin(int kernel_id, hipStream_t stream)
{
    if (!g_trace_on || !((g_trace_mask >> kernel_id) & 1ull)) return;
    g_pending_start = get_event();
    if (g_pending_start) (void)hipEventRecord(g_pending_start, stream);
}

void trace_end(int kernel_id, hipStream_t stream)
{
    if (!g_trace_on || !g_pending_start) return;
    hipEvent_t e1 = get_event();
    if (!e1) { g_event_pool.push_back(g_pending_start); g_pending_start = nullptr; return; }
    (void)hipEventRecord(e1, stream);
    g_trace_recs.push_back(TraceRec{kernel_id, g_pending_start, e1});
    g_pending_start = nullptr;
}

namespace {

// ------------------------------------------------------------------------------------------------
// validation helpers
constexpr int64_t MAX_ELEMS = (int64_t)1 << 31;

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline size_t esize(int dtype) { return dtype == DORA_F32 ? 4 : 2; }
inline bool is16(int dtype) { return dtype != DORA_F32; }
inline int dt_of(int dtype) { return dtype == DORA_F16 ? DT_F16 : DT_BF16; }
inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

dora_status check_desc(const dora_desc* d, bool need_weights)
{
    if (!d) return DORA_ERR_NULL;
    if (d->dtype != DORA_F32 && d->dtype != DORA_BF16 && d->dtype != DORA_F16) return DORA_ERR_DTYPE;
    const int64_t mult = is16(d->dtype) ? 8 : 4;
    if (d->d_out < mult || d->d_out % mult) return DORA_ERR_SHAPE;
    if (d->tokens < 0) return DORA_ERR_SHAPE;
    if (d->tokens * d->d_out >= MAX_ELEMS) return DORA_ERR_SHAPE;
    if (need_weights) {
        if (d->d_in < mult || d->d_in % mult) return DORA_ERR_SHAPE;
        if (d->r < mult || d->r % mult) return DORA_ERR_SHAPE;
        if (d->d_out * d->d_in >= MAX_ELEMS || d->tokens * d->d_in >= MAX_ELEMS) return DORA_ERR_SHAPE;
        if (d->r * d->d_in >= MAX_ELEMS || d->d_out * d->r >= MAX_ELEMS || d->tokens * d->r >= MAX_ELEMS)
            return DORA_ERR_SHAPE;
    }
    if (!(d->s == d->s) || !(d->eps == d->eps)) return DORA_ERR_SHAPE;  // NaN scalars
    return DORA_OK;
}

inline float eff_eps(const dora_desc* d) { return d->eps > 0.f ? d->eps : (is16(d->dtype) ? 1e-6f : 1e-12f); }

#define DORA_REQ_PTR(p)                          \
    do {                                         \
        if (!(p)) return DORA_ERR_NULL;          \
        if (!aligned((p), 16)) return DORA_ERR_ALIGN; \
    } while (0)
#define DORA_OPT_PTR(p)                                \
    do {                                               \
        if ((p) && !aligned((p), 16)) return DORA_ERR_ALIGN; \
    } while (0)
#define DORA_HIP(call)                                 \
    do {                                               \
        if ((call) != hipSuccess) return DORA_ERR_HIP; \
    } while (0)

// ------------------------------------------------------------------------------------------------
// workspace layout: a bump allocator over the caller's scratch, every block 256-byte aligned
struct Bump {
    char* base;
    size_t off;
    explicit Bump(void* p) : base(static_cast<char*>(p)), off(0) {}
    template <typename T> T* take(size_t count)
    {
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += up256(count * sizeof(T));
        return p;
    }
    void* take_bytes(size_t bytes)
    {
        void* p = base ? base + off : nullptr;
        off += up256(bytes);
        return p;
    }
};

constexpr int TILE = 128;
inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct NormPlan {
    int tiles_n;   // N tiles of the [d_out, r] row-dot contractions
    int ks_u;      // split of d_in for U = W A^T
    int ks_g;      // split of d_in for G = A A^T
    // 16-bit path of higher ranks
    float *base_p, *cross_p, *ba_p, *gram_p;
    bf16_t *Ghi, *Glo;
    // where the three sums come from one launch (16-bit up to NORM_ROWS_MAX_RANK, fp32)
    int slices, tiles_per_slice;   // of the columns
    int row_blocks;                // fp32: of 16 rows to a workgroup
    float* part;                   // [3][slices][d_out]
};

// Split-K factors of the two norm contractions, which share a launch: 256 CUs x two 128x128-tile workgroups hold 512 at a
// time.  `fit` and `room` fill one round.  The cost counted, in K steps of 64: rounds of cross-term slices, each its K steps
// plus about six for what comes before the first and for the row-dot epilogue; the Gram workgroups, last in the launch, are
// beside them where slots are left, at their own length, and a round of their own where not.  The cheapest split is taken
// if it promises a seventh or more (smaller promises measured as losses: 5120 x 27648, r 384, seven slices 169 us against
// 157 for four).  Measured over weight sets of 1.2 GB in turn, us of a norm, one round -> this: 27648 x 5120, r 384 224 -> 191
// (648 tiles: two rounds, the second a quarter full); 14336 x 4096, r 768 203 -> 185; 4096 x 14336, r 384 92 -> 82 and
// 3072 x 6000, r 512 72 -> 59 (long Gram slices ended last); 8192 x 8192, r 128 55.6 -> 53.8 (no slot left for the Gram tiles).
// The Gram partials stay within 8 MiB where the split of the cross term alone asks for more of them.  Whether a shape's
// scratch fits the static array does not depend on the choice: (fit, room) decides, the others must agree.
size_t norm_split_bytes(int64_t d_out, int64_t r, int tiles_n, int ks_u, int ks_g)
{
    return up256((size_t)ks_u * d_out * 4) + up256((size_t)ks_u * tiles_n * d_out * 4) + up256((size_t)tiles_n * d_out * 4) +
           up256((size_t)ks_g * r * r * 4) + 2 * up256((size_t)r * r * 2);
}
void norm_split(int64_t d_out, int64_t d_in, int64_t r, int& ks_u, int& ks_g)
{
    // 64 bits: the tiles of G alone number up to (2^28 / TILE)^2
    const int64_t tiles_n = (r + TILE - 1) / TILE, tiles_u = (d_out + TILE - 1) / TILE * tiles_n, tiles_g = tiles_n * tiles_n;
    const int64_t ktiles = (d_in + 63) / 64;
    const int64_t fit = std::max<int64_t>(1, std::min<int64_t>({512 / tiles_u, 8, ktiles}));
    const int64_t left = 512 - tiles_u * fit;
    const int64_t room = std::max<int64_t>(1, std::min<int64_t>({(left > 0 ? left : 512) / tiles_g, 16, ktiles}));
    const int64_t most = std::max<int64_t>(1, (8 << 20) / (4 * r * r));
    auto fits_static = [&](int64_t ks, int64_t kg) {
        return norm_split_bytes(d_out, r, (int)tiles_n, (int)ks, (int)kg) <= DORA_STATIC_SCRATCH_BYTES;
    };
    auto cost = [&](int64_t ks, int64_t kg) {
        const int64_t rounds = (tiles_u * ks + 511) / 512, slots = rounds * 512 - tiles_u * ks;
        const int64_t steps_u = (ktiles + ks - 1) / ks, steps_g = (ktiles + kg - 1) / kg;
        const int64_t own = tiles_g * kg > slots ? steps_g + 6 : std::max<int64_t>(0, steps_g - steps_u);
        return rounds * (steps_u + 6) + own;
    };
    int64_t best_u = fit, best_g = room, best = cost(fit, room) * 6 / 7;
    const bool fits = fits_static(fit, room);
    for (int64_t ks = 1; ks <= std::min<int64_t>(8, ktiles); ++ks) {
        const int64_t kg = std::max(room, std::min(ks, most));
        if (cost(ks, kg) <= best && fits_static(ks, kg) == fits) { best = cost(ks, kg) - 1; best_u = ks; best_g = kg; }
    }
    ks_u = (int)best_u;
    ks_g = (int)best_g;
}

// Slices of the columns for the launch that forms the three sums (norm_rows.hip): the cheapest in rounds of workgroups, two
// to a CU up to r 128, one beyond, counted in cycles of a tile (its share of reading W, or its MFMAs) and of what comes before
// the first.
void norm_slices(int64_t d_out, int64_t d_in, int64_t r, size_t fixed_bytes, size_t most_bytes, int& slices, int& tiles_per_slice)
{
    const int64_t blocks = (d_out + TILE - 1) / TILE, tiles = (d_in + TILE - 1) / TILE;
    const int64_t at_once = r <= 128 ? 512 : 256, tile = r <= 128 ? 6600 : std::max<int64_t>((r + 63) / 64 * 850 + 600, 3300), first = 8000;
    int64_t best = -1;
    for (int64_t n = 1; n <= std::min<int64_t>(64, tiles) && (n == 1 || blocks * n <= 4096); ++n) {
        const int64_t per = (tiles + n - 1) / n, used = (tiles + per - 1) / per;
        const int64_t cost = (blocks * used + at_once - 1) / at_once * (per * tile + first);
        if (n > 1 && fixed_bytes + up256((size_t)3 * used * d_out * 4) > most_bytes) break;
        if (best < 0 || cost < best) { best = cost; slices = (int)used; tiles_per_slice = (int)per; }
    }
}

// fp32 norm: rows of a workgroup (one or two blocks of 16) and slices of the columns, the cheapest in tenths of a microsecond.  A
// CU has one workgroup of sixteen waves; a wave takes groups of 32 columns, and 64 of the rank take it 1 us (1.6 with 32 rows) with
// a SIMD to itself and 3.5 (5.9) where four share one; with 16 rows it takes the rank in pieces of 64, whose last one costs two
// thirds where it holds 32 or less, with 32 rows in pieces of 32.  A round of workgroups costs 1.9 more, and 5 where the slices
// have to be added.  (16 rows, and slices only where they filled CUs without any: 5120 x 27648, r 768 4764 us, 320 workgroups in
// two rounds, 2464 now, 1280 in five; 8192 x 8192, r 384 711 -> 595, where 16 rows read A from the L2 twice as often; 512 x 512, r
// 512 32 -> 16; 2048 x 2048, r 128 26 -> 23; 1000 x 772, r 36 stays at 10.  88 shapes: 0.6 % from the best of 22 choices.)
void norm_f32_shape(int64_t d_out, int64_t d_in, int64_t r, int& row_blocks, int& slices)
{
    static const int cost_of[2][5] = {{0, 10, 18, 27, 35}, {0, 16, 29, 43, 59}};   // of 64 ranks, by waves on a SIMD
    const uint32_t groups = (uint32_t)(d_in + 31) / 32, blocks = (uint32_t)(d_out + 15) / 16;   // (each below 2^31 / 4)
    const uint32_t most = std::max<uint32_t>(1, std::min<uint32_t>({(uint32_t)r / 3, groups, 32}));   // r / 3: the scratch
    int64_t best = -1;
    for (uint32_t rb = 1; rb <= 2; ++rb) {
        const int64_t sixths = rb == 2 ? (r + 31) / 32 * 3 : r / 64 * 6 + (r % 64 == 0 ? 0 : r % 64 <= 32 ? 4 : 6);
        for (uint32_t n = 1; n <= most; ++n) {
            const uint32_t per = (groups + n - 1) / n, rounds = ((blocks + rb - 1) / rb * n + 255) / 256;
            const int64_t walk = (int64_t)(per / 16) * cost_of[rb - 1][4] + cost_of[rb - 1][(per % 16 + 3) / 4];
            const int64_t cost = rounds * (walk * sixths / 6 + 19) + (n > 1 ? 50 : 0);
            if (best < 0 || cost < best) { best = cost; row_blocks = (int)rb; slices = (int)n; }
        }
    }
}

void plan_norm(const dora_desc* d, Bump& b, NormPlan& n)
{
    memset(&n, 0, sizeof(n));
    n.tiles_n = cdiv(d->r, TILE);
    if (is16(d->dtype)) {
        const Bump start = b;
        norm_split(d->d_out, d->d_in, d->r, n.ks_u, n.ks_g);
        n.base_p = b.take<float>((size_t)n.ks_u * d->d_out);
        n.cross_p = b.take<float>((size_t)n.ks_u * n.tiles_n * d->d_out);
        n.ba_p = b.take<float>((size_t)n.tiles_n * d->d_out);
        n.gram_p = b.take<float>((size_t)n.ks_g * d->r * d->r);
        n.Ghi = b.take<bf16_t>((size_t)d->r * d->r);
        n.Glo = b.take<bf16_t>((size_t)d->r * d->r);
        if (d->r > NORM_ROWS_MAX_RANK) return;
        // One launch: its partial sums and, where the caller asks for G, the slices of the Gram matrix take the place of all
        // of these.  Which shapes fit the static array stays as the split above has it.
        const size_t gram = up256((size_t)n.ks_g * d->r * d->r * 4);
        norm_slices(d->d_out, d->d_in, d->r, gram, std::max<size_t>(b.off - start.off, DORA_STATIC_SCRATCH_BYTES), n.slices, n.tiles_per_slice);
        Bump o = start;
        n.part = o.take<float>((size_t)3 * n.slices * d->d_out);
        n.gram_p = o.take<float>((size_t)n.ks_g * d->r * d->r);
        b.off = std::max(b.off, o.off);
    } else {
        norm_f32_shape(d->d_out, d->d_in, d->r, n.row_blocks, n.slices);
        // Scratch of d_out (2 r) + r^2 floats, three blocks, whatever the sums need of it (3 slices d_out): which shapes fit the static
        // array does not change with the slices.
        n.part = b.take<float>((size_t)d->d_out * d->r);
        b.off += up256((size_t)d->r * d->r * 4) + up256((size_t)d->d_out * d->r * 4);
    }
}

// Split of K for the products with a 16-bit output of at most 256 tiles of 128 x 128: h = x A^T and dh = s dz B over [tokens,
// r], x W^T and dz W of short batches; ldb: row length of the N-side operand.  K is cut into slices (fp32 partials in the workspace,
// summed in slice order by a small reduce launch), as many as are cheapest in twentieths of a microsecond: for each K step of 64 of
// a slice 8 while every workgroup has a CU to itself and 15 where two share one, with a weight of 2 MB and more 9 and 17 (10 and 19
// where its rows do not start at lines of 128 bytes), one more while K is whole (there three), when too few loads are in flight for
// what comes from memory; 100 for the reduce launch, and the partials written and read at 3.4 TB/s.  At most two workgroups per CU,
// 16 slices, and two K steps to a slice at least.  (Forward, us with weights from memory / left in a cache: 512 tokens, 4096 x
// 4096, r 64 with K whole 57 / 43, in two slices 51 / 44; 256 tokens, 3000 x 2056 46 / 29, in three 36 / 32; 512 tokens, 4096 x 4104
// 72 / 58, in two 58 / 57.  247 forwards and backwards of 65 to 2048 tokens are within 0.9 % of the best number of slices with
// weights from memory and 0.5 % in a cache, those with rows off the lines 1.4 % and 1.0 %.  x A^T of 512 tokens, K 4096, r 64 in one
// slice 11.9 us, 7.2 in 16; of 4096 tokens, r 384, in two slices and in five, K 4096 42 and 48 us, 14336 106 and 94, 27648 181 and
// 156.)
// saves: what K whole would save beside, where the product could share a launch with others (a launch and a round of its own, 10 us:
// step of 2048 x 2048, r 64, 512 tokens 75 us with all gradients in one launch, 84 with dx in slices).
constexpr int64_t SHARED_LAUNCH_SAVES = 200;
inline int product_ksplit(int dtype, int64_t M, int64_t N, int64_t K, int64_t ldb, int64_t saves = 0)
{
    if (!is16(dtype) || M <= 0) return 1;
    const int64_t tiles = ((M + TILE - 1) / TILE) * ((N + TILE - 1) / TILE), steps = (K + 63) / 64;
    if (tiles > 256) return 1;
    const bool weight = N * K >= 1 << 20, off = weight && ldb % 64 != 0;   // (a factor of less is in a cache whenever it is used)
    const int64_t alone = off ? 10 : weight ? 9 : 8, shared = off ? 19 : weight ? 17 : 15, whole = alone + (off ? 3 : 1);
    int64_t best = 1, least = whole * steps;
    for (int64_t ks = 2; ks <= std::min<int64_t>({512 / tiles, 16, steps / 2}); ++ks) {
        const int64_t cost = (tiles * ks > 256 ? shared : alone) * ((steps + ks - 1) / ks) + 100 + saves + ks * M * N / 21000;
        if (cost < least) { least = cost; best = ks; }
    }
    return (int)best;
}

// ------------------------------------------------------------------------------------------------
// one contraction, either dtype
struct Seg { const void* a; int64_t lda; const void* b; int64_t ldb; int K; };

GemmArgs bf16_args(int dt, bool a_kc, bool b_kc, int M, int N, const Seg* segs, int nseg, float alpha, void* c,
                   int64_t ldc, bool c_f32, int tag)
{
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    for (int i = 0; i < nseg; ++i)
        g.seg[i] = GemmSeg{(const bf16_t*)segs[i].a, (const bf16_t*)segs[i].b, segs[i].lda, segs[i].ldb, segs[i].K};
    g.nseg = nseg; g.M = M; g.N = N; g.a_kcontig = a_kc; g.b_kcontig = b_kc;
    g.epilogue = c_f32 ? EPI_STORE_F32 : EPI_STORE_BF16;
    g.alpha = alpha; g.c = c; g.ldc = ldc; g.ksplit = 1; g.tag = tag; g.dt = dt;
    return g;
}

SgemmArgs f32_args(bool a_kc, bool b_kc, int M, int N, const Seg* segs, int nseg, float alpha, void* c, int64_t ldc)
{
    SgemmArgs g;
    memset(&g, 0, sizeof(g));
    for (int i = 0; i < nseg; ++i)
        g.seg[i] = SgemmSeg{(const float*)segs[i].a, (const float*)segs[i].b, segs[i].lda, segs[i].ldb, segs[i].K, false};
    g.nseg = nseg; g.M = M; g.N = N; g.a_kcontig = a_kc; g.b_kcontig = b_kc; g.alpha = alpha; g.c = (float*)c; g.ldc = ldc;
    return g;
}

// One 16-bit product; skp != nullptr: scratch for the K slices, the product is then split as product_ksplit says and the
// reduce launch does what the epilogue (EPI_STORE_BF16 or EPI_COMPOSE) would have done.
// waiting: see Waiting; a product that is not split leaves it as it is.
hipError_t launch_product(const GemmArgs& g, int trace_id, float* skp, hipStream_t st, Waiting* waiting = nullptr)
{
    const int ks = (skp && g.ldc == g.N) ? product_ksplit(DORA_BF16, g.M, g.N, g.seg[0].K, g.seg[0].ldb) : 1;
    if (ks <= 1) return launch_gemm_bf16(g, trace_id, st);
    const bool compose = g.epilogue == EPI_COMPOSE;
    GemmArgs p = g;
    p.epilogue = EPI_STORE_F32; p.c = skp; p.ksplit = ks; p.c2 = nullptr;
    hipError_t e = launch_gemm_bf16(p, trace_id, st);
    if (e != hipSuccess) return e;
    return launch_splitk_reduce(skp, ks, (int64_t)g.M * g.N, g.dt == DT_F16 ? DORA_F16 : DORA_BF16, g.c, compose ? 1.f : g.alpha2,
                                g.c2, st, compose ? g.colscale : nullptr, g.colbias, g.N, waiting);
}

// skp != nullptr (16-bit outputs): scratch for the K slices of the first segment.  c2 / alpha2: optional second output
// alpha2 * (A B^T) (16-bit storage only).
hipError_t contract(int dtype, bool a_kc, bool b_kc, int M, int N, const Seg* segs, int nseg, float alpha, void* c,
                    int64_t ldc, bool c_f32, int trace_id, hipStream_t st, float* skp = nullptr, void* c2 = nullptr,
                    float alpha2 = 0.f, Waiting* waiting = nullptr)
{
    if (is16(dtype)) {
        const int tag = (trace_id == DORA_K_GEMM_LORA || trace_id == DORA_K_GEMM_DB) ? 1 : 0;
        GemmArgs g = bf16_args(dt_of(dtype), a_kc, b_kc, M, N, segs, nseg, alpha, c, ldc, c_f32, tag);
        g.c2 = c2; g.alpha2 = alpha2;
        return launch_product(g, trace_id, c_f32 ? nullptr : skp, st, waiting);
    }
    const SgemmArgs g = f32_args(a_kc, b_kc, M, N, segs, nseg, alpha, c, ldc);
    return launch_f32(&g, 1, nullptr, nullptr, nullptr, trace_id, st);
}

// ------------------------------------------------------------------------------------------------
// factored norm (Sec. 2, Algorithm 1)
// base_sq != nullptr: the base term of Eq. 2 comes from the caller's cache and W is not squared again
// c == nullptr: only the terms are wanted.  terms != nullptr: [3, d_out] fp32 receives base_sq, cross, ba_sq.
// G_out != nullptr: [r, r] fp32 receives the Gram matrix of Eq. 4.
// waiting != nullptr: the last launch may be left there.
// Eq. 6 riding on the norm's last launch: set `done` when g / gm1 were written there
struct MagOut { const float* m; float eps; float* g; float* gm1; bool done; };

dora_status norm_impl(const dora_desc* d, const void* W, const void* A, const void* B, float* c, const NormPlan& n,
                      hipStream_t st, const float* base_sq = nullptr, float* terms = nullptr, float* G_out = nullptr,
                      MagOut* mag = nullptr, Waiting* waiting = nullptr)
{
    const int d_out = (int)d->d_out, d_in = (int)d->d_in, r = (int)d->r;
    if (d->s == 0.f) {  // scale-is-zero fast path: no U, no G
        if (terms) {  // base_sq from W (or the cache), cross = ba_sq = 0, G not formed
            if (G_out) DORA_HIP(launch_gram_reduce(nullptr, 0, r, G_out, nullptr, nullptr, DT_BF16, st));  // zero partials: G = 0
            if (!base_sq && is16(d->dtype)) {
                DORA_HIP(launch_rownorm_s0_16((const bf16_t*)W, dt_of(d->dtype), n.base_p, d_out, d_in, true, st));
                base_sq = n.base_p;
            }
            if (base_sq) DORA_HIP(launch_norm_final(norm_final_args(base_sq, 1, nullptr, 0, nullptr, 0, 0.0, c, terms, d_out), st));
            else DORA_HIP(launch_rownorm_f32((const float*)W, c, terms, d_out, d_in, false, st));
            return DORA_OK;
        }
        if (base_sq) DORA_HIP(launch_norm_final(norm_final_args(base_sq, 1, nullptr, 0, nullptr, 0, 0.0, c, nullptr, d_out), st));
        else if (is16(d->dtype)) DORA_HIP(launch_rownorm_s0_16((const bf16_t*)W, dt_of(d->dtype), c, d_out, d_in, false, st));
        else DORA_HIP(launch_rownorm_f32((const float*)W, c, nullptr, d_out, d_in, false, st));
        return DORA_OK;
    }
    if (is16(d->dtype)) {
        if ((int64_t)r * r >= MAX_ELEMS) return DORA_ERR_SHAPE;   // G is an operand of the B G product
        const int dt = dt_of(d->dtype);
        // past that rank B no longer fits the registers of a workgroup
        if (r <= NORM_ROWS_MAX_RANK) {
            const NormRowsArgs a{(const bf16_t*)W, (const bf16_t*)A, (const bf16_t*)B, d_out, d_in, r, n.slices, n.tiles_per_slice, n.part};
            DORA_HIP(launch_norm_rows(a, dt, st));
            if (G_out) {
                Seg sg{A, d_in, A, d_in, d_in};
                GemmArgs g = bf16_args(dt, true, true, r, r, &sg, 1, 1.f, n.gram_p, r, true, 0);
                g.ksplit = n.ks_g;
                DORA_HIP(launch_gemm_bf16(g, DORA_K_GRAM, st));
                DORA_HIP(launch_gram_reduce(n.gram_p, n.ks_g, r, G_out, nullptr, nullptr, dt, st));
            }
            const size_t all = (size_t)n.slices * d_out;
            const NormFinalArgs fin = norm_final_args(base_sq ? base_sq : n.part, base_sq ? 1 : n.slices, n.part + all, n.slices,
                                                      n.part + 2 * all, n.slices, (double)d->s, c, terms, d_out, mag ? mag->m : nullptr,
                                                      mag ? mag->eps : 0.f, mag ? mag->g : nullptr, mag ? mag->gm1 : nullptr);
            if (waiting) { waiting->norm = true; waiting->norm_args = fin; }
            else DORA_HIP(launch_norm_final(fin, st));
            if (mag) mag->done = true;
            return DORA_OK;
        }
        GemmArgs g;
        // cross term (Eq. 3) and base term: U = W A^T tile by tile, reduced against B in registers
        memset(&g, 0, sizeof(g));
        g.seg[0] = GemmSeg{(const bf16_t*)W, (const bf16_t*)A, d_in, d_in, d_in};
        g.nseg = 1; g.M = d_out; g.N = r; g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_ROWDOT; g.alpha = 1.f; g.dt = dt;
        g.ksplit = n.ks_u; g.rowdot = (const bf16_t*)B; g.ld_rowdot = r; g.rowdot_partial = n.cross_p;
        g.base_sq_partial = base_sq ? nullptr : n.base_p;
        // Gram matrix (Eq. 4): split-K partials, then a fixed-order sum and the hi/lo 16-bit expansion.  It is
        // independent of the cross term and far too small to fill the chip, so its workgroups ride in the same launch.
        GemmArgs gg;
        memset(&gg, 0, sizeof(gg));
        gg.seg[0] = GemmSeg{(const bf16_t*)A, (const bf16_t*)A, d_in, d_in, d_in};
        gg.nseg = 1; gg.M = r; gg.N = r; gg.a_kcontig = 1; gg.b_kcontig = 1; gg.epilogue = EPI_STORE_F32; gg.alpha = 1.f;
        gg.dt = dt; gg.c = n.gram_p; gg.ldc = r; gg.ksplit = n.ks_g;
        DORA_HIP(launch_gemm_bf16_pair(g, gg, DORA_K_NORM_CROSS, st));
        DORA_HIP(launch_gram_reduce(n.gram_p, n.ks_g, r, G_out, n.Ghi, n.Glo, dt, st));
        // BA-norm term: rowdot(B, B G) with G = Ghi + Glo kept to ~16 mantissa bits (G is symmetric,
        // so G serves as its own K-contiguous N-side operand)
        memset(&g, 0, sizeof(g));
        g.seg[0] = GemmSeg{(const bf16_t*)B, n.Ghi, r, r, r};
        g.seg[1] = GemmSeg{(const bf16_t*)B, n.Glo, r, r, r};
        g.nseg = 2; g.M = d_out; g.N = r; g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_ROWDOT; g.alpha = 1.f; g.dt = dt;
        g.ksplit = 1; g.rowdot = (const bf16_t*)B; g.ld_rowdot = r; g.rowdot_partial = n.ba_p; g.tag = 1;
        DORA_HIP(launch_gemm_bf16(g, DORA_K_BA_SQ, st));
        DORA_HIP(launch_norm_final(norm_final_args(base_sq ? base_sq : n.base_p, base_sq ? 1 : n.ks_u, n.cross_p, n.ks_u * n.tiles_n,
                                                   n.ba_p, n.tiles_n, (double)d->s, c, terms, d_out, mag ? mag->m : nullptr,
                                                   mag ? mag->eps : 0.f, mag ? mag->g : nullptr, mag ? mag->gm1 : nullptr), st));
        if (mag) mag->done = true;
        return DORA_OK;
    }
    const NormF32Args a{(const float*)W, (const float*)A, (const float*)B, d_out, d_in, r, base_sq, (float)(2.0 * d->s),
                        (float)((double)d->s * d->s), c, terms, mag ? mag->m : nullptr, mag ? mag->eps : 0.f,
                        mag ? mag->g : nullptr, mag ? mag->gm1 : nullptr, n.slices, n.part, n.row_blocks};
    DORA_HIP(launch_norm_f32(a, st));
    const size_t all = (size_t)n.slices * d_out;
    if (n.slices > 1)
        DORA_HIP(launch_norm_final(norm_final_args(base_sq ? base_sq : n.part, base_sq ? 1 : n.slices, n.part + all, n.slices,
                                                   n.part + 2 * all, n.slices, (double)d->s, c, terms, d_out, a.m, a.eps, a.g, a.gm1), st));
    if (mag) mag->done = true;
    if (G_out) {
        Seg sg{A, d_in, A, d_in, d_in};
        DORA_HIP(contract(DORA_F32, true, true, r, r, &sg, 1, 1.f, G_out, r, true, DORA_K_GRAM, st));
    }
    return DORA_OK;
}

// ------------------------------------------------------------------------------------------------
// forward / backward plans
struct FwdPlan {
    NormPlan norm;
    float *c, *g, *gm1;
    void *h, *lora, *hs, *base_a;
    float* skp;   // K slices of h = xa A^T, then of x W^T (nullptr: neither is split)
};
// Forward of a few tokens in 16-bit storage: two launches that stream the weights (few_tokens.hip) instead of tiles, where
// they are the faster ones.  Every workgroup of the second launch first sums h and multiplies it with its rows of B, which
// costs tokens times rank whatever d_in is, and beyond 16384 rows of W its workgroups need a second round.  Measured with
// weights and inputs rotated through 600 MB, time against the tiles' (one_product: the K-concatenated product):
//   up to 16384 rows: 4096 x 4096, r 384, 1 token 20 us / 36, 64 tokens 34 / 40; 17 to 32 tokens 0.85 to 1.1 at r 1536, up
//     to 1.1 beyond; 33 to 64 tokens 0.78 to 0.96 at r 640, 0.92 to 1.09 at 768 (the upper half past 48 tokens),
//     1.2 to 1.4 at 1536 (8192 x 2048, r 2048, 64 tokens 78 us / 54)
//   beyond: up to 16 tokens 0.5 to 0.9 up to r 2048 (past 32768 rows 0.9 to 1.0 at 1024, 1.1 at 1536); 17 to 32 tokens 0.8 to
//     1.03 up to r 256, 1.0 to 1.1 at 384, and up to 1.2 for d_in 8192; 33 to 64 tokens 0.8 to 1.0 up to r 128 for d_in 2048
//     to 4096, 1.0 to 1.3 for shorter rows (27648 x 5120, r 384, 64 tokens 112 us / 96)
// Base, lora and a compose pass are slower tiles, so against those the lines lie further out: 0.8 to 0.95 at r 1024 and 64
// tokens, and beyond 16384 rows up to 16 tokens 0.4 to 1.05, 32 tokens 0.7 to 1.0 at r 384, 64 tokens 0.8 to 1.0 at r 256.
inline bool few_tokens(const dora_desc* d, bool one_product)
{
    const int64_t T = d->tokens, r = d->r;
    if (!is16(d->dtype) || T <= 0 || T > FEW_TOKENS_MAX) return false;
    if (d->d_out <= 16384) {
        if (T <= 32) return T <= 16 || !one_product || r <= 1536;
        return r <= (one_product ? (T <= 48 ? 768 : 640) : 1024);
    }
    if (T <= 16) return !one_product || r <= (d->d_out <= 32768 ? 2048 : 1024);
    if (T <= 32) return r <= (one_product ? 256 : 512) && d->d_in <= 5120;
    return one_product ? r <= 128 && d->d_in >= 2048 && d->d_in <= 4096 : r <= 256 && d->d_in <= 4096;
}

// scratch for the K slices of a [tokens, n] product over k whose N-side operand has rows of ldb
inline size_t slice_floats(const dora_desc* d, int64_t n, int64_t k, int64_t ldb)
{
    const int ks = product_ksplit(d->dtype, d->tokens, n, k, ldb);
    return ks > 1 ? (size_t)ks * d->tokens * n : 0;
}

void plan_fwd(const dora_desc* d, Bump& b, FwdPlan& p, bool need_norm, bool need_h, bool need_lora,
              bool need_hs = false, bool need_base_a = false)
{
    memset(&p, 0, sizeof(p));
    if (need_norm) plan_norm(d, b, p.norm);
    p.c = b.take<float>((size_t)d->d_out);
    p.g = b.take<float>((size_t)d->d_out);
    p.gm1 = b.take<float>((size_t)d->d_out);
    if (need_h) p.h = b.take_bytes((size_t)d->tokens * d->r * esize(d->dtype));
    if (need_lora) p.lora = b.take_bytes((size_t)d->tokens * d->d_out * esize(d->dtype));
    if (need_hs) p.hs = b.take_bytes((size_t)d->tokens * d->r * esize(d->dtype));
    if (need_base_a) p.base_a = b.take_bytes((size_t)d->tokens * d->d_out * esize(d->dtype));
    // (where the K-concatenated product gives way to few_tokens, the compose pass does too)
    size_t slices = few_tokens(d, false) ? (size_t)few_tokens_h_slices(d->tokens, d->r, d->d_in) * d->tokens * d->r : 0;
    slices = std::max({slices, slice_floats(d, d->r, d->d_in, d->d_in), slice_floats(d, d->d_out, d->d_in, d->d_in)});
    if (slices) p.skp = b.take<float>(slices);
}

struct BwdPlan {
    NormPlan norm;
    float *c, *g, *gm1, *dm_partial;
    void *dz, *dh, *h, *inner, *dzb;
    float* skp;   // K slices of whichever product is under way (nullptr: none is split)
};
void plan_bwd(const dora_desc* d, Bump& b, BwdPlan& p, bool need_norm, bool need_h, bool need_inner,
              bool need_dzb = false)
{
    memset(&p, 0, sizeof(p));
    if (need_norm) plan_norm(d, b, p.norm);
    p.c = b.take<float>((size_t)d->d_out);
    p.g = b.take<float>((size_t)d->d_out);
    p.gm1 = b.take<float>((size_t)d->d_out);
    p.dm_partial = b.take<float>((size_t)compose_bwd_slabs(d->tokens, (int)d->d_out, d->dtype) * d->d_out);
    p.dz = b.take_bytes((size_t)d->tokens * d->d_out * esize(d->dtype));
    p.dh = b.take_bytes((size_t)d->tokens * d->r * esize(d->dtype));
    if (need_h) p.h = b.take_bytes((size_t)d->tokens * d->r * esize(d->dtype));
    if (need_inner) p.inner = b.take_bytes((size_t)d->tokens * d->d_out * esize(d->dtype));
    if (need_dzb) p.dzb = b.take_bytes((size_t)d->tokens * d->d_out * esize(d->dtype));
    size_t slices = std::max(slice_floats(d, d->r, d->d_out, d->r), slice_floats(d, d->d_in, d->d_out, d->d_in));
    if (need_h) slices = std::max(slices, slice_floats(d, d->r, d->d_in, d->d_in));
    if (need_inner) slices = std::max(slices, slice_floats(d, d->d_out, d->d_in, d->d_in));
    if (slices) p.skp = b.take<float>(slices);
}

dora_status check_ws(void* ws, size_t ws_bytes, size_t need)
{
    if (need == 0) return DORA_OK;
    if (!ws) return DORA_ERR_NULL;
    if (!aligned(ws, 256)) return DORA_ERR_ALIGN;
    if (ws_bytes < need) return DORA_ERR_WORKSPACE;
    return DORA_OK;
}

// base = x W^T, h = x A^T, lora = h B^T (App. A item 1; lora == nullptr: not that one)
// xa: the adapter branch's input (x itself unless LoRA dropout gives that branch an input of its own)
dora_status forward_contractions(const dora_desc* d, const void* x, const void* W, const void* A, const void* B,
                                 void* base, void* h, void* lora, hipStream_t st, const void* xa = nullptr,
                                 float* skp = nullptr, Waiting* waiting = nullptr)
{
    const int T = (int)d->tokens, d_out = (int)d->d_out, d_in = (int)d->d_in, r = (int)d->r;
    Seg s0{x, d_in, W, d_in, d_in};
    Seg s1{xa ? xa : x, d_in, A, d_in, d_in};
    // (16-bit: base and h are NOT paired into one launch: h's extra tiles would form a fifth, nearly empty
    // round behind the four full rounds of 256 x 256 base tiles and cost more than a launch of their own)
    // (h after base, not before: it then finds part of x still in the memory-side cache; the other order costs 10 us)
    if (d->dtype == DORA_F32) {
        const SgemmArgs g[2] = {f32_args(true, true, T, d_out, &s0, 1, 1.f, base, d_out), f32_args(true, true, T, r, &s1, 1, 1.f, h, r)};
        DORA_HIP(launch_f32(g, 2, nullptr, nullptr, nullptr, DORA_K_GEMM_BASE, st));
    } else {
        DORA_HIP(contract(d->dtype, true, true, T, d_out, &s0, 1, 1.f, base, d_out, false, DORA_K_GEMM_BASE, st, skp, nullptr, 0.f, waiting));
        DORA_HIP(contract(d->dtype, true, true, T, r, &s1, 1, 1.f, h, r, false, DORA_K_GEMM_H, st, skp, nullptr, 0.f, waiting));
    }
    if (!lora) return DORA_OK;
    Seg s2{h, r, B, r, r};
    DORA_HIP(contract(d->dtype, true, true, T, d_out, &s2, 1, 1.f, lora, d_out, false, DORA_K_GEMM_LORA, st));
    return DORA_OK;
}

// fp32: lora = h B^T composed in its own launch; y holds base and receives y, inner (may be nullptr)
hipError_t f32_lora_composed(const dora_desc* d, const void* h, const void* B, const float* g, const float* gm1, const void* bias,
                             void* y, void* inner, hipStream_t st)
{
    const int T = (int)d->tokens, d_out = (int)d->d_out, r = (int)d->r;
    Seg s2{h, r, B, r, r};
    SgemmArgs a = f32_args(true, true, T, d_out, &s2, 1, 1.f, y, d_out);
    a.composed = 1; a.g = g; a.gm1 = gm1; a.bias = (const float*)bias; a.s = d->s; a.inner = (float*)inner;
    return launch_f32(&a, 1, nullptr, nullptr, nullptr, DORA_K_GEMM_LORA, st);
}

// y = g (.) (x W^T + s (x A^T) B^T) (+ bias) of a few tokens; c: the row norm (g is formed in the last launch)
dora_status forward_few_tokens(const dora_desc* d, const void* x, const void* W, const void* A, const void* B, const float* m,
                               const float* c, const void* bias, void* y, void* saved_h, void* saved_inner, float* h_part,
                               hipStream_t st)
{
    FewTokensArgs a;
    memset(&a, 0, sizeof(a));
    a.x = (const bf16_t*)x; a.T = (int)d->tokens; a.K = (int)d->d_in;
    a.w = (const bf16_t*)A; a.N = (int)d->r;
    a.ksplit = a.h_slices = few_tokens_h_slices(d->tokens, d->r, d->d_in);
    a.part = h_part;
    DORA_HIP(launch_few_tokens_h(a, dt_of(d->dtype), st));
    a.w = (const bf16_t*)W; a.N = (int)d->d_out; a.ksplit = 1;
    a.h_part = h_part; a.r = (int)d->r; a.b = (const bf16_t*)B;
    a.s = d->s; a.eps = eff_eps(d); a.m = m; a.c = c; a.bias = (const bf16_t*)bias;
    a.y = (bf16_t*)y; a.inner = (bf16_t*)saved_inner; a.h_out = (bf16_t*)saved_h;
    DORA_HIP(launch_few_tokens_y(a, dt_of(d->dtype), st));
    return DORA_OK;
}

}  // namespace
}  // namespace dora

using namespace dora;

// ================================================================================================
extern "C" {

const char* dora_status_str(int status)
{
    switch (status) {
        case DORA_OK: return "ok";
        case DORA_ERR_NULL: return "required pointer is NULL";
        case DORA_ERR_SHAPE: return "invalid shape or scalar";
        case DORA_ERR_ALIGN: return "pointer not sufficiently aligned";
        case DORA_ERR_DTYPE: return "unknown dtype";
        case DORA_ERR_WORKSPACE: return "workspace too small";
        case DORA_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

size_t dora_workspace_bytes(const dora_desc* desc, int phase)
{
    if (phase == DORA_PHASE_COMPOSE_BACKWARD) {
        if (check_desc(desc, false) != DORA_OK) return 0;
        const size_t n = up256((size_t)compose_bwd_slabs(desc->tokens, (int)desc->d_out, desc->dtype) * desc->d_out * sizeof(float));
        return n > 0 ? n : 256;   // 0 is reserved for "invalid desc"
    }
    if (check_desc(desc, true) != DORA_OK) return 0;
    Bump b(nullptr);
    switch (phase) {
        case DORA_PHASE_NORM: { NormPlan n; plan_norm(desc, b, n); break; }
        case DORA_PHASE_FORWARD: { FwdPlan p; plan_fwd(desc, b, p, true, true, true, true); break; }
        case DORA_PHASE_BACKWARD: { BwdPlan p; plan_bwd(desc, b, p, false, false, false); break; }
        case DORA_PHASE_BACKWARD_RECOMPUTE: { BwdPlan p; plan_bwd(desc, b, p, true, true, true); break; }
        case DORA_PHASE_FORWARD_DROPOUT: { FwdPlan p; plan_fwd(desc, b, p, true, true, true, true, true); break; }
        case DORA_PHASE_BACKWARD_DROPOUT: { BwdPlan p; plan_bwd(desc, b, p, true, true, true, true); break; }
        default: return 0;
    }
    return b.off > 0 ? b.off : 256;
}

dora_status dora_norm(const dora_desc* desc, const void* W, const void* A, const void* B, float* w_norm, void* ws,
                      size_t ws_bytes, void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(w_norm);
    Bump sizing(nullptr);
    NormPlan n;
    plan_norm(desc, sizing, n);
    if ((st = check_ws(ws, ws_bytes, sizing.off)) != DORA_OK) return st;
    Bump b(ws);
    plan_norm(desc, b, n);
    return norm_impl(desc, W, A, B, w_norm, n, (hipStream_t)stream);
}

size_t dora_norm_static_max_bytes(void) { return DORA_STATIC_SCRATCH_BYTES; }

dora_status dora_norm_static(const dora_desc* desc, const void* W, const void* A, const void* B, float* w_norm,
                             void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(w_norm);
    Bump sizing(nullptr);
    NormPlan n;
    plan_norm(desc, sizing, n);
    if (sizing.off > DORA_STATIC_SCRATCH_BYTES) return DORA_ERR_WORKSPACE;  // shape beyond the static scratch
    void* ptr = static_scratch_ptr();
    if (!ptr) return DORA_ERR_HIP;
    // every partial the norm kernels read back is written in full by the launch before it, so nothing
    // left in the array by an earlier call (of any shape) needs clearing
    Bump b(ptr);
    plan_norm(desc, b, n);
    return norm_impl(desc, W, A, B, w_norm, n, (hipStream_t)stream);
}

dora_status dora_base_sq(const dora_desc* desc, const void* W, float* base_sq, void* stream)
{
    dora_status st = check_desc(desc, false);
    if (st != DORA_OK) return st;
    const int64_t mult = is16(desc->dtype) ? 8 : 4;
    if (desc->d_in < mult || desc->d_in % mult || desc->d_out * desc->d_in >= MAX_ELEMS) return DORA_ERR_SHAPE;
    DORA_REQ_PTR(W); DORA_REQ_PTR(base_sq);
    const int d_out = (int)desc->d_out, d_in = (int)desc->d_in;
    hipStream_t s = (hipStream_t)stream;
    if (is16(desc->dtype)) DORA_HIP(launch_rownorm_s0_16((const bf16_t*)W, dt_of(desc->dtype), base_sq, d_out, d_in, true, s));
    else DORA_HIP(launch_rownorm_f32((const float*)W, base_sq, nullptr, d_out, d_in, true, s));
    return DORA_OK;
}

dora_status dora_norm_cached(const dora_desc* desc, const float* base_sq, const void* W, const void* A, const void* B,
                             float* w_norm, void* ws, size_t ws_bytes, void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(base_sq); DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(w_norm);
    Bump sizing(nullptr);
    NormPlan n;
    plan_norm(desc, sizing, n);
    if ((st = check_ws(ws, ws_bytes, sizing.off)) != DORA_OK) return st;
    Bump b(ws);
    plan_norm(desc, b, n);
    return norm_impl(desc, W, A, B, w_norm, n, (hipStream_t)stream, base_sq);
}

dora_status dora_norm_terms(const dora_desc* desc, const void* W, const void* A, const void* B, float* terms, float* G,
                            void* ws, size_t ws_bytes, void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(terms);
    DORA_OPT_PTR(G);
    Bump sizing(nullptr);
    NormPlan n;
    plan_norm(desc, sizing, n);
    if ((st = check_ws(ws, ws_bytes, sizing.off)) != DORA_OK) return st;
    Bump b(ws);
    plan_norm(desc, b, n);
    return norm_impl(desc, W, A, B, nullptr, n, (hipStream_t)stream, nullptr, terms, G);
}

dora_status dora_norm_assemble(const dora_desc* desc, const float* terms, float* w_norm, void* stream)
{
    dora_status st = check_desc(desc, false);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(terms); DORA_REQ_PTR(w_norm);
    const int d_out = (int)desc->d_out;
    // the same kernel, and so the same arithmetic in the same order, as the last step of dora_norm
    DORA_HIP(launch_norm_final(norm_final_args(terms, 1, terms + d_out, 1, terms + 2 * (size_t)d_out, 1, (double)desc->s, w_norm,
                                               nullptr, d_out), (hipStream_t)stream));
    return DORA_OK;
}

dora_status dora_mag_scale(const dora_desc* desc, const float* m, const float* w_norm, float* g, float* gm1,
                           void* stream)
{
    dora_status st = check_desc(desc, false);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(m); DORA_REQ_PTR(w_norm);
    if (!g && !gm1) return DORA_ERR_NULL;
    DORA_OPT_PTR(g); DORA_OPT_PTR(gm1);
    DORA_HIP(launch_mag_scale(m, w_norm, eff_eps(desc), g, gm1, (int)desc->d_out, (hipStream_t)stream));
    return DORA_OK;
}

dora_status dora_compose(const dora_desc* desc, const void* base, const void* lora, const float* g, const float* gm1,
                         void* out, int write_delta, void* inner, void* stream)
{
    dora_status st = check_desc(desc, false);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(base); DORA_REQ_PTR(lora); DORA_REQ_PTR(g); DORA_REQ_PTR(out);
    DORA_OPT_PTR(gm1); DORA_OPT_PTR(inner);
    DORA_HIP(launch_compose_fwd(desc->dtype, base, lora, g, gm1, nullptr, desc->s, out, write_delta ? 1 : 0, inner, desc->tokens,
                                (int)desc->d_out, (hipStream_t)stream));
    return DORA_OK;
}

dora_status dora_compose_backward(const dora_desc* desc, const void* dy, const void* inner, const float* g,
                                  const float* w_norm, void* dz, float* dm, void* ws, size_t ws_bytes, void* stream)
{
    dora_status st = check_desc(desc, false);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(dy); DORA_REQ_PTR(g); DORA_REQ_PTR(dz);
    DORA_OPT_PTR(dm);
    float* partial = nullptr;
    if (dm) {
        DORA_REQ_PTR(inner); DORA_REQ_PTR(w_norm);
        size_t need = up256((size_t)compose_bwd_slabs(desc->tokens, (int)desc->d_out, desc->dtype) * desc->d_out * sizeof(float));
        if ((st = check_ws(ws, ws_bytes, need)) != DORA_OK) return st;
        partial = (float*)ws;
    }
    hipStream_t s = (hipStream_t)stream;
    DORA_HIP(launch_compose_bwd(desc->dtype, dy, inner, g, nullptr, dz, nullptr, partial, desc->tokens, (int)desc->d_out, s));
    if (dm)
        DORA_HIP(launch_dm_final(DmFinalArgs{partial, compose_bwd_slabs(desc->tokens, (int)desc->d_out, desc->dtype), w_norm,
                                             eff_eps(desc), dm, (int)desc->d_out}, s));
    return DORA_OK;
}

dora_status dora_project(const dora_desc* desc, const void* x, const void* W, const void* A, const void* B,
                         void* base, void* h, void* lora, void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(x); DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B);
    DORA_REQ_PTR(base); DORA_REQ_PTR(h); DORA_REQ_PTR(lora);
    if (desc->tokens == 0) return DORA_OK;
    return forward_contractions(desc, x, W, A, B, base, h, lora, (hipStream_t)stream);
}

// inner = x W^T + s h B^T as one K-concatenated product  [x | s h] [W | B]^T, hs = s h; the caller sets epilogue and outputs
static GemmArgs inner_product(const dora_desc* d, const void* x, const void* W, const void* B, const void* hs)
{
    const int T = (int)d->tokens, d_out = (int)d->d_out, d_in = (int)d->d_in, r = (int)d->r;
    Seg segs[2] = {{x, d_in, W, d_in, d_in}, {hs, r, B, r, r}};
    return bf16_args(dt_of(d->dtype), true, true, T, d_out, segs, 2, 1.f, nullptr, d_out, false, 0);
}

// one_product: the K-concatenated forward (h, then [x | s h] [W | B]^T with the compose in its epilogue), else x W^T,
// h B^T and a compose pass over both.
static dora_status forward_impl(const dora_desc* desc, const void* x, const void* x_lora, const void* W, const void* A,
                                const void* B, const float* m, const float* w_norm, const void* bias, void* y, void* saved_h,
                                void* saved_inner, float* w_norm_out, void* ws, size_t ws_bytes, void* stream, bool one_product)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(m);
    if (desc->tokens > 0) { DORA_REQ_PTR(x); DORA_REQ_PTR(y); }
    DORA_OPT_PTR(x_lora);
    DORA_OPT_PTR(w_norm); DORA_OPT_PTR(bias); DORA_OPT_PTR(saved_h); DORA_OPT_PTR(saved_inner); DORA_OPT_PTR(w_norm_out);
    const bool need_norm = (w_norm == nullptr);
    const bool dropout = (x_lora != nullptr);
    const bool f32_plain = desc->dtype == DORA_F32 && !dropout;
    const bool need_lora = !one_product && !f32_plain && saved_inner == nullptr;
    Bump sizing(nullptr);
    FwdPlan p;
    plan_fwd(desc, sizing, p, need_norm, saved_h == nullptr, need_lora, one_product, dropout);
    if ((st = check_ws(ws, ws_bytes, sizing.off)) != DORA_OK) return st;
    Bump b(ws);
    plan_fwd(desc, b, p, need_norm, saved_h == nullptr, need_lora, one_product, dropout);
    hipStream_t s = (hipStream_t)stream;
    const int T = (int)desc->tokens, d_out = (int)desc->d_out, d_in = (int)desc->d_in, r = (int)desc->r;

    float* const gm1 = one_product ? nullptr : p.gm1;   // only the compose pass reads g - 1
    MagOut mag{m, eff_eps(desc), p.g, gm1, false};
    const float* c = w_norm;
    Waiting waiting;          // Eq. 5 and 6: g is read by the last launch of the tiled routes only
    const bool streamed = !dropout && few_tokens(desc, one_product);
    if (need_norm) {
        float* cw = w_norm_out ? w_norm_out : p.c;
        if ((st = norm_impl(desc, W, A, B, cw, p.norm, s, nullptr, nullptr, nullptr, &mag, T > 0 && !streamed ? &waiting : nullptr)) != DORA_OK)
            return st;
        c = cw;
    } else if (w_norm_out && w_norm_out != w_norm) {
        DORA_HIP(hipMemcpyAsync(w_norm_out, w_norm, sizeof(float) * d_out, hipMemcpyDeviceToDevice, s));
    }
    if (T == 0) return DORA_OK;
    if (streamed)
        return forward_few_tokens(desc, x, W, A, B, m, c, bias, y, saved_h, saved_inner, p.skp, s);
    if (!mag.done) DORA_HIP(launch_mag_scale(m, c, eff_eps(desc), p.g, gm1, d_out, s));
    void* h = saved_h ? saved_h : p.h;
    if (one_product) {
        // h = x A^T, written twice from the same accumulators: as it is (the saved tensor) and scaled by s
        Seg s1{x, d_in, A, d_in, d_in};
        DORA_HIP(contract(desc->dtype, true, true, T, r, &s1, 1, 1.f, h, r, false, DORA_K_GEMM_H, s, p.skp, p.hs, desc->s, &waiting));
        DORA_HIP(launch_waiting(waiting, s));
        GemmArgs g = inner_product(desc, x, W, B, p.hs);
        g.epilogue = EPI_COMPOSE;
        g.c = y;
        g.colscale = p.g;
        g.colbias = (const bf16_t*)bias;
        g.c2 = saved_inner;
        DORA_HIP(launch_product(g, DORA_K_GEMM_FUSED_FWD, p.skp, s));
        return DORA_OK;
    }
    if (f32_plain) {
        if ((st = forward_contractions(desc, x, W, A, B, y, h, nullptr, s)) != DORA_OK) return st;
        DORA_HIP(launch_waiting(waiting, s));
        DORA_HIP(f32_lora_composed(desc, h, B, p.g, p.gm1, bias, y, saved_inner, s));
        return DORA_OK;
    }
    // base lands in y and lora in the inner buffer; the compose pass then runs in place on both
    void* lora = saved_inner ? saved_inner : p.lora;
    Seg sx{x, d_in, W, d_in, d_in}, sa{x_lora, d_in, W, d_in, d_in};
    if (dropout && is16(desc->dtype) && product_ksplit(desc->dtype, T, d_out, d_in, d_in, SHARED_LAUNCH_SAVES) == 1) {
        // x W^T and x_lora W^T in one launch where their tiles fill rounds better together (2056 x 3000, 1501 tokens: 204 of 128 x
        // 128 each, one to a CU: 69 us in two launches, 56 in one)
        const int dt = dt_of(desc->dtype);
        const GemmArgs g0 = bf16_args(dt, true, true, T, d_out, &sx, 1, 1.f, y, d_out, false, 0);
        const GemmArgs g1 = bf16_args(dt, true, true, T, d_out, &sa, 1, 1.f, p.base_a, d_out, false, 0);
        if (gemm_bf16_pairs(g0, g1)) {
            DORA_HIP(launch_gemm_bf16_pair(g0, g1, DORA_K_GEMM_BASE, s));
            Seg s1{x_lora, d_in, A, d_in, d_in}, s2{h, r, B, r, r};
            DORA_HIP(contract(desc->dtype, true, true, T, r, &s1, 1, 1.f, h, r, false, DORA_K_GEMM_H, s, p.skp, nullptr, 0.f, &waiting));
            DORA_HIP(contract(desc->dtype, true, true, T, d_out, &s2, 1, 1.f, lora, d_out, false, DORA_K_GEMM_LORA, s));
            DORA_HIP(launch_waiting(waiting, s));
            DORA_HIP(launch_compose_fwd(desc->dtype, p.base_a, lora, p.g, p.gm1, bias, desc->s, y, 2, saved_inner, T, d_out, s));
            return DORA_OK;
        }
    }
    if ((st = forward_contractions(desc, x, W, A, B, y, h, lora, s, x_lora, p.skp, &waiting)) != DORA_OK) return st;
    DORA_HIP(launch_waiting(waiting, s));
    if (!dropout) {
        DORA_HIP(launch_compose_fwd(desc->dtype, y, lora, p.g, p.gm1, bias, desc->s, y, 0, saved_inner, T, d_out, s));
        return DORA_OK;
    }
    // LoRA dropout: the compose runs on the adapter branch's own base x_lora W^T and its delta is added to
    // the frozen layer's output already in y
    DORA_HIP(contract(desc->dtype, true, true, T, d_out, &sa, 1, 1.f, p.base_a, d_out, false, DORA_K_GEMM_BASE, s, p.skp));
    DORA_HIP(launch_compose_fwd(desc->dtype, p.base_a, lora, p.g, p.gm1, bias, desc->s, y, 2, saved_inner, T, d_out, s));
    return DORA_OK;
}

// bf16 takes the K-concatenated product: one rounding where base, lora and the compose pass had three, and no pass over
// [tokens, d_out] beside the product (8192 x 8192, r 384, 8192 tokens, forward and backward: 2089 -> 2021 us; 4096 x 4096,
// 4096 tokens, forward: 216 -> 191 us; 27648 x 5120 and back with recompute: 13.79 -> 12.93 ms).  fp16 keeps the compose
// pass: s h is rounded to storage before the product, and fp16's exponent range does not hold s h wherever it holds h.
static bool forward_in_one_product(const dora_desc* d) { return d && d->dtype == DORA_BF16; }

dora_status dora_forward(const dora_desc* desc, const void* x, const void* W, const void* A, const void* B,
                         const float* m, const float* w_norm, const void* bias, void* y, void* saved_h, void* saved_inner,
                         float* w_norm_out, void* ws, size_t ws_bytes, void* stream)
{
    return forward_impl(desc, x, nullptr, W, A, B, m, w_norm, bias, y, saved_h, saved_inner, w_norm_out, ws, ws_bytes, stream,
                        forward_in_one_product(desc));
}

dora_status dora_forward_dropout(const dora_desc* desc, const void* x, const void* x_lora, const void* W, const void* A,
                                 const void* B, const float* m, const float* w_norm, const void* bias, void* y,
                                 void* saved_h, void* saved_inner, float* w_norm_out, void* ws, size_t ws_bytes,
                                 void* stream)
{
    if (desc && desc->tokens > 0 && !x_lora) return DORA_ERR_NULL;
    // dropout switched off (evaluation): the adapter's input is x itself, so x W^T serves both branches
    if (desc && desc->tokens > 0 && x_lora == x) x_lora = nullptr;
    return forward_impl(desc, x, x_lora, W, A, B, m, w_norm, bias, y, saved_h, saved_inner, w_norm_out, ws, ws_bytes, stream,
                        !x_lora && forward_in_one_product(desc));
}

dora_status dora_forward_fused(const dora_desc* desc, const void* x, const void* W, const void* A, const void* B,
                               const float* m, const float* w_norm, const void* bias, void* y, void* saved_h, void* saved_inner,
                               float* w_norm_out, void* ws, size_t ws_bytes, void* stream)
{
    if (check_desc(desc, true) == DORA_OK && !is16(desc->dtype)) return DORA_ERR_DTYPE;
    return forward_impl(desc, x, nullptr, W, A, B, m, w_norm, bias, y, saved_h, saved_inner, w_norm_out, ws, ws_bytes, stream,
                        true);
}

// fp32, plain module, in two launches: dh and the first stage of dm's column sum, then dx, dA, dB and its second stage.  dz = g
// (.) dy is not written: g goes into the operands as they are read (formed on the way, and for the second launch, where only
// the norm is there), into dB as its rows are stored.  (compose backward, column
// sum, dh, dx and dA with dB as launches of their own: a pass over [tokens, d_out] and three launches more.)
static dora_status backward_f32(const dora_desc* d, const void* dy, const void* x, const void* W, const void* A, const void* B,
                                RowScale g, const float* c, const void* h, const void* inner, void* dx, float* dA, float* dB,
                                float* dm, float* dm_partial, float* g_buf, void* dh, hipStream_t s)
{
    const int T = (int)d->tokens, d_out = (int)d->d_out, d_in = (int)d->d_in, r = (int)d->r;
    SgemmArgs q[3];
    int n = 0;
    if (dx || dA) {
        Seg sh{dy, d_out, B, r, d_out};
        q[n] = f32_args(true, false, T, r, &sh, 1, d->s, dh, r);
        if (g.m && f32_tiled(q[0])) {                  // tiles do not form it: a launch of its own, 4 us beside 50 and more
            DORA_HIP(launch_mag_scale(g.m, g.g, g.eps, g_buf, nullptr, d_out, s));
            g = RowScale{g_buf, nullptr, 0.f};
        }
        q[n].seg[0].scaled = true; q[n++].ascale = g;
    }
    const ColumnSum sum{(const float*)dy, (const float*)inner, T, d_out, dm_partial};
    const ScaleOut form{g, g_buf, d_out};
    DORA_HIP(launch_f32(q, n, dm && T > 0 ? &sum : nullptr, nullptr, g.m ? &form : nullptr, DORA_K_GEMM_DH, s));
    if (g.m) g = RowScale{g_buf, nullptr, 0.f};
    n = 0;
    if (dx) {
        Seg sx[2] = {{dy, d_out, W, d_in, d_out}, {dh, r, A, d_in, r}};
        q[n] = f32_args(true, false, T, d_in, sx, 2, 1.f, dx, d_in);
        q[n].seg[0].scaled = true; q[n++].ascale = g;
    }
    Seg sa{dh, r, x, d_in, T}, sb{dy, d_out, h, r, T};
    if (dA) q[n++] = f32_args(false, false, r, d_in, &sa, 1, 1.f, dA, d_in);
    if (dB) {
        q[n] = f32_args(false, false, d_out, r, &sb, 1, d->s, dB, r);
        if (T > 0) q[n].rowscale = g;
        ++n;
    }
    const ColumnFinal fin{dm_partial, column_sum_slabs(T), c, eff_eps(d), dm, d_out};
    DORA_HIP(launch_f32(q, n, nullptr, dm ? &fin : nullptr, nullptr, DORA_K_GEMM_DX, s));
    return DORA_OK;
}

// x_lora == nullptr: the plain module (dx = dz W + dh A).  Otherwise the adapter branch has its own input:
// dx = dy W (frozen path; x itself is not needed), dx_lora = ((g-1) dy) W + dh A, dA and the recomputed
// h / inner come from x_lora.
static dora_status backward_impl(const dora_desc* desc, const void* dy, const void* x, const void* x_lora, const void* W,
                                 const void* A, const void* B, const float* m, const float* w_norm, const void* saved_h,
                                 const void* saved_inner, void* dx, void* dx_lora, float* dA, float* dB, float* dm,
                                 void* ws, size_t ws_bytes, void* stream)
{
    dora_status st = check_desc(desc, true);
    if (st != DORA_OK) return st;
    const bool dropout = (x_lora != nullptr);
    const void* xa = dropout ? x_lora : x;
    DORA_REQ_PTR(W); DORA_REQ_PTR(A); DORA_REQ_PTR(B); DORA_REQ_PTR(m);
    if (desc->tokens > 0) { DORA_REQ_PTR(dy); DORA_REQ_PTR(xa); }
    DORA_OPT_PTR(w_norm); DORA_OPT_PTR(saved_h); DORA_OPT_PTR(saved_inner);
    DORA_OPT_PTR(dx); DORA_OPT_PTR(dx_lora); DORA_OPT_PTR(dA); DORA_OPT_PTR(dB); DORA_OPT_PTR(dm);
    const bool need_norm = (w_norm == nullptr);
    const bool need_inner = (dm != nullptr) && (saved_inner == nullptr);
    const bool need_h = (saved_h == nullptr) && (dB != nullptr || need_inner);
    const bool need_dzb = dropout && (dx_lora != nullptr);
    Bump sizing(nullptr);
    BwdPlan p;
    plan_bwd(desc, sizing, p, need_norm, need_h, need_inner, need_dzb);
    if ((st = check_ws(ws, ws_bytes, sizing.off)) != DORA_OK) return st;
    Bump b(ws);
    plan_bwd(desc, b, p, need_norm, need_h, need_inner, need_dzb);
    hipStream_t s = (hipStream_t)stream;
    const int T = (int)desc->tokens, d_out = (int)desc->d_out, d_in = (int)desc->d_in, r = (int)desc->r;
    const int dt = desc->dtype;

    MagOut mag{m, eff_eps(desc), p.g, p.gm1, false};
    const float* c = w_norm;
    Waiting waiting;          // Eq. 5 and 6 up to the first reader of g, dm's second stage up to the end
    if (need_norm) {
        if ((st = norm_impl(desc, W, A, B, p.c, p.norm, s, nullptr, nullptr, nullptr, &mag, &waiting)) != DORA_OK) return st;
        c = p.c;
    }
    const bool mag_in_compose = !mag.done && !need_inner;   // then the compose backward is the only reader of g
    if (!mag.done && !mag_in_compose) DORA_HIP(launch_mag_scale(m, c, eff_eps(desc), p.g, p.gm1, d_out, s));

    const void* h = saved_h;
    const void* inner = saved_inner;
    if (T > 0 && need_inner && !saved_h && forward_in_one_product(desc)) {
        // recompute (gradient-checkpointing pattern) as the forward forms it; s h waits in the dh buffer
        Seg s1{xa, d_in, A, d_in, d_in};
        DORA_HIP(contract(dt, true, true, T, r, &s1, 1, 1.f, p.h, r, false, DORA_K_GEMM_H, s, p.skp, p.dh, desc->s, &waiting));
        GemmArgs g = inner_product(desc, xa, W, B, p.dh);
        g.c = p.inner;
        DORA_HIP(launch_product(g, DORA_K_GEMM_FUSED_FWD, p.skp, s));
        inner = p.inner;
        h = p.h;
    } else if (T > 0 && need_inner) {
        DORA_HIP(launch_waiting(waiting, s));
        // base -> dz buffer, lora -> inner buffer, then inner = s*lora + base in place; the dz buffer is overwritten
        // by dz afterwards
        void* const lora = dt == DORA_F32 ? nullptr : p.inner;
        if (saved_h) {
            Seg s0{xa, d_in, W, d_in, d_in};
            DORA_HIP(contract(dt, true, true, T, d_out, &s0, 1, 1.f, p.dz, d_out, false, DORA_K_GEMM_BASE, s, p.skp));
            Seg s2{saved_h, r, B, r, r};
            if (lora) DORA_HIP(contract(dt, true, true, T, d_out, &s2, 1, 1.f, lora, d_out, false, DORA_K_GEMM_LORA, s));
        } else {
            if ((st = forward_contractions(desc, xa, W, A, B, p.dz, p.h, lora, s, nullptr, p.skp)) != DORA_OK) return st;
            h = p.h;
        }
        if (lora) DORA_HIP(launch_compose_fwd(dt, p.dz, p.inner, p.g, p.gm1, nullptr, desc->s, nullptr, 0, p.inner, T, d_out, s));
        else DORA_HIP(f32_lora_composed(desc, h, B, p.g, p.gm1, nullptr, p.dz, p.inner, s));
        inner = p.inner;
    } else if (T > 0 && need_h) {
        Seg s1{xa, d_in, A, d_in, d_in};
        DORA_HIP(contract(dt, true, true, T, r, &s1, 1, 1.f, p.h, r, false, DORA_K_GEMM_H, s, p.skp, nullptr, 0.f, &waiting));
        h = p.h;
    }
    DORA_HIP(launch_waiting(waiting, s));

    // Launches that share the outputs' writes with the reads of dy, W and A are left to callers who keep those apart: dx, dx_lora
    // or a gradient may lie over dy (or a weight that is not needed again) where each is written after its last reader.
    struct Span { const void* p; size_t bytes; };
    const size_t e = esize(dt), grad_dA = (size_t)r * d_in * 4, grad_dB = (size_t)d_out * r * 4;
    const Span in_dy{dy, (size_t)T * d_out * e}, in_W{W, (size_t)d_out * d_in * e}, in_A{A, (size_t)r * d_in * e};
    const Span out_dx{dx, (size_t)T * d_in * e}, out_dxl{dx_lora, (size_t)T * d_in * e}, out_dA{dA, grad_dA}, out_dB{dB, grad_dB},
        out_dm{dm, (size_t)d_out * 4};
    auto over = [](const Span& o, const Span& i) {
        const uintptr_t a = (uintptr_t)o.p, b = (uintptr_t)i.p;
        return a && b && a < b + i.bytes && b < a + o.bytes;
    };
    auto over_inputs = [&](const Span& o) { return over(o, in_dy) || over(o, in_W) || over(o, in_A); };
    const bool weights_apart = !over_inputs(out_dA) && !over_inputs(out_dB);
    if (dt == DORA_F32 && !dropout && weights_apart && !over_inputs(out_dx) && !over_inputs(out_dm))
        return backward_f32(desc, dy, xa, W, A, B, mag_in_compose ? RowScale{c, m, eff_eps(desc)} : RowScale{p.g, nullptr, 0.f}, c, h,
                            inner, dx, dA, dB, dm, p.dm_partial, p.g, p.dh, s);

    // compose backward: dz = g*dy (and (g-1)*dy for a separate adapter input) and the fused two-stage column
    // reduction for dm
    DORA_HIP(launch_compose_bwd(dt, dy, inner, mag_in_compose ? c : p.g, p.gm1, p.dz, need_dzb ? p.dzb : nullptr,
                                dm ? p.dm_partial : nullptr, T, d_out, s, mag_in_compose ? m : nullptr, eff_eps(desc)));
    if (dm) {
        waiting.dm = true;
        waiting.dm_args = DmFinalArgs{p.dm_partial, compose_bwd_slabs(T, d_out, dt), c, eff_eps(desc), dm, d_out};
    }

    // dh = s * dz B   (gradient reaching h)
    if ((dropout ? dx_lora : dx) || dA) {
        Seg sh{p.dz, d_out, B, r, d_out};
        DORA_HIP(contract(dt, true, false, T, r, &sh, 1, desc->s, p.dh, r, false, DORA_K_GEMM_DH, s, p.skp, nullptr, 0.f, &waiting));
    }
    DORA_HIP(launch_waiting(waiting, s));
    // dx = dz W + dh A : one contraction over the concatenated K range.  With dropout the frozen path, dx = dy W, and the adapter
    // path, dx_lora = ((g-1) dy) W + dh A
    Seg sx[2] = {{dropout ? p.dzb : p.dz, d_out, W, d_in, d_out}, {p.dh, r, A, d_in, r}};
    Seg sf{dy, d_out, W, d_in, d_out};
    void* const dx_sum = dropout ? dx_lora : dx;
    Seg sa{p.dh, r, xa, d_in, T};  // dA = dh^T xa
    Seg sb{p.dz, d_out, h, r, T};  // dB = s * dz^T h
    // 16-bit, K not in slices: both input gradients in one launch where their tiles fill rounds better together (2056 x 3000,
    // 1501 tokens: 288 of 128 x 128 each, one and an eighth to a CU; together 144 of 256 x 256: 77 us in two launches, 59 in
    // one), and the weight gradients with them where CUs are left for those
    bool paired = false;
    if (is16(dt) && T > 0 && product_ksplit(dt, T, d_in, d_out, d_in, SHARED_LAUNCH_SAVES) == 1) {
        GemmArgs in[2], wg[2];
        int n = 0, nw = 0;
        if (dropout && dx) in[n++] = bf16_args(dt_of(dt), true, false, T, d_in, &sf, 1, 1.f, dx, d_in, false, 0);
        if (dx_sum) in[n++] = bf16_args(dt_of(dt), true, false, T, d_in, sx, 2, 1.f, dx_sum, d_in, false, 0);
        if (dA) wg[nw++] = bf16_args(dt_of(dt), false, false, r, d_in, &sa, 1, 1.f, dA, d_in, true, 0);
        if (dB) wg[nw++] = bf16_args(dt_of(dt), false, false, d_out, r, &sb, 1, desc->s, dB, r, true, 0);
        paired = n == 2 && !over_inputs(out_dxl) && gemm_bf16_pairs(in[0], in[1]);
        if ((n == 1 || paired) && weights_apart && gemm_bf16_grads_together(in, n, wg, nw)) {
            DORA_HIP(launch_gemm_bf16_grads(in, n, wg, nw, DORA_K_GEMM_DX, s));
            return DORA_OK;
        }
        if (paired) DORA_HIP(launch_gemm_bf16_pair(in[0], in[1], DORA_K_GEMM_DX, s));
    }
    if (!paired) {
        if (dropout && dx) DORA_HIP(contract(dt, true, false, T, d_in, &sf, 1, 1.f, dx, d_in, false, DORA_K_GEMM_DX, s, p.skp));
        if (dx_sum) DORA_HIP(contract(dt, true, false, T, d_in, sx, 2, 1.f, dx_sum, d_in, false, DORA_K_GEMM_DX, s, p.skp));
    }
    if (dA && dB && is16(dt)) {
        // the two weight gradients are independent and individually too small to fill the chip: one launch
        GemmArgs ga = bf16_args(dt_of(dt), false, false, r, d_in, &sa, 1, 1.f, dA, d_in, true, 0);
        GemmArgs gb = bf16_args(dt_of(dt), false, false, d_out, r, &sb, 1, desc->s, dB, r, true, 0);
        DORA_HIP(launch_gemm_bf16_pair(ga, gb, DORA_K_GEMM_DA, s));
    } else if (dA && dB) {
        const SgemmArgs q[2] = {f32_args(false, false, r, d_in, &sa, 1, 1.f, dA, d_in), f32_args(false, false, d_out, r, &sb, 1, desc->s, dB, r)};
        DORA_HIP(launch_f32(q, 2, nullptr, nullptr, nullptr, DORA_K_GEMM_DA, s));
    } else {
        if (dA) DORA_HIP(contract(dt, false, false, r, d_in, &sa, 1, 1.f, dA, d_in, true, DORA_K_GEMM_DA, s));
        if (dB) DORA_HIP(contract(dt, false, false, d_out, r, &sb, 1, desc->s, dB, r, true, DORA_K_GEMM_DB, s));
    }
    return DORA_OK;
}

dora_status dora_backward(const dora_desc* desc, const void* dy, const void* x, const void* W, const void* A,
                          const void* B, const float* m, const float* w_norm, const void* saved_h,
                          const void* saved_inner, void* dx, float* dA, float* dB, float* dm, void* ws,
                          size_t ws_bytes, void* stream)
{
    return backward_impl(desc, dy, x, nullptr, W, A, B, m, w_norm, saved_h, saved_inner, dx, nullptr, dA, dB, dm, ws, ws_bytes,
                         stream);
}

dora_status dora_backward_dropout(const dora_desc* desc, const void* dy, const void* x_lora, const void* W, const void* A,
                                  const void* B, const float* m, const float* w_norm, const void* saved_h,
                                  const void* saved_inner, void* dx, void* dx_lora, float* dA, float* dB, float* dm,
                                  void* ws, size_t ws_bytes, void* stream)
{
    if (desc && desc->tokens > 0 && !x_lora) return DORA_ERR_NULL;
    if (desc && desc->tokens == 0 && !x_lora) x_lora = W;  // nothing of it is read; keeps the dropout code path
    return backward_impl(desc, dy, nullptr, x_lora, W, A, B, m, w_norm, saved_h, saved_inner, dx, dx_lora, dA, dB, dm, ws,
                         ws_bytes, stream);
}

dora_status dora_probe_copy(const void* src, void* dst, size_t bytes, void* stream)
{
    DORA_REQ_PTR(src); DORA_REQ_PTR(dst);
    if (bytes % 16) return DORA_ERR_SHAPE;
    DORA_HIP(launch_copy_probe(src, dst, bytes, (hipStream_t)stream));
    return DORA_OK;
}

dora_status dora_probe_mfma(const void* operands, float* sink, int iters, int workgroups, void* stream)
{
    DORA_REQ_PTR(operands); DORA_REQ_PTR(sink);
    if (iters < 0 || workgroups < 0 || workgroups > 65536) return DORA_ERR_SHAPE;
    DORA_HIP(launch_mfma_probe(operands, sink, iters, workgroups, (hipStream_t)stream));
    return DORA_OK;
}

// ------------------------------------------------------------------------------------------------
void dora_trace_enable(int on) { g_trace_on = (on != 0); }

void dora_trace_select(uint64_t kernel_mask) { g_trace_mask = kernel_mask; }

void dora_trace_reset(void)
{
    for (auto& r : g_trace_recs) { g_event_pool.push_back(r.e0); g_event_pool.push_back(r.e1); }
    g_trace_recs.clear();
    for (int i = 0; i < DORA_K_COUNT; ++i) { g_trace_ms[i] = 0.0; g_trace_n[i] = 0; }
}

int dora_trace_collect(void)
{
    int rc = DORA_OK;
    for (auto& r : g_trace_recs) {
        float ms = 0.f;
        if (hipEventSynchronize(r.e1) != hipSuccess || hipEventElapsedTime(&ms, r.e0, r.e1) != hipSuccess) rc = DORA_ERR_HIP;
        else if (r.id >= 0 && r.id < DORA_K_COUNT) { g_trace_ms[r.id] += ms; g_trace_n[r.id] += 1; }
        g_event_pool.push_back(r.e0);
        g_event_pool.push_back(r.e1);
    }
    g_trace_recs.clear();
    return rc;
}

int dora_trace_get(int kernel_id, double* total_ms, int64_t* launches)
{
    if (kernel_id < 0 || kernel_id >= DORA_K_COUNT) return DORA_ERR_SHAPE;
    if (total_ms) *total_ms = g_trace_ms[kernel_id];
    if (launches) *launches = g_trace_n[kernel_id];
    return DORA_OK;
}

const char* dora_trace_name(int kernel_id)
{
    static const char* names[DORA_K_COUNT] = {
        "norm_cross_WAt", "gram_AAt", "gram_reduce", "ba_sq_BGB", "norm_final", "mag_scale", "gemm_base_xWt",
        "gemm_h_xAt", "gemm_lora_hBt", "compose_fwd", "compose_bwd", "dm_final", "gemm_dh_dzB", "gemm_dx",
        "gemm_dA", "gemm_dB", "probe_copy", "probe_mfma", "gemm_fused_fwd", "splitk_reduce"};
    return (kernel_id >= 0 && kernel_id < DORA_K_COUNT) ? names[kernel_id] : "?";
}

}  // extern "C"
