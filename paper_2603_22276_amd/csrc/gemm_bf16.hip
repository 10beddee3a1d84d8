// 16-bit (bf16 or fp16 storage) MFMA GEMM family for gfx950 (CDNA4), fp32 accumulation.
//
//   C[M,N] = alpha * sum_seg sum_k Aop[m,k] * Bop[n,k]
//
// One kernel template serves every dense contraction of the DoRA module: x W^T, x A^T, h B^T
// (both operands K-contiguous), dz W + dh A and dz B (N-side operand K-strided), dh^T x and dz^T h
// (both K-strided), and the factored-norm products of Sec. 2: U = W A^T with the row-dot epilogue
// of Eq. 3 (U never leaves registers), G = A A^T (Eq. 4, split-K partials), and rowdot(B, B G).
//
// Structure (per workgroup): a BM x BN tile of C; K is walked in steps of 64 through rings of LDS
// buffers that the global loads fill directly (buffer_load ... lds, 16 bytes per lane, no register
// staging).  A K step of 64 makes every row segment a load instruction fetches a full 128-byte line;
// 64-byte segments stream at about two thirds of that rate.  Four 64-wide wavefronts per workgroup,
// each owning a (BM/2) x (BN/2) sub-tile.  The N-side fragment is fed as the MFMA's first operand so
// that every lane ends up holding four consecutive n for one m, which makes the epilogue's stores and
// row-dots vector-friendly.  Workgroup ids are remapped so that each of the 8 XCDs (own L2 each) works
// on a compact block of tiles, walked in groups of 8 tile-rows.
//
// Two tile shapes.  128 x 128 (64 x 64 per wave as 2 x 2 of v_mfma_f32_32x32x16, two workgroups per CU,
// which hide each other's stalls) for the skinny products.  256 x 256 (128 x 128 per wave as 8 x 8 of
// v_mfma_f32_16x16x32, accumulators in AGPRs, one wave per SIMD, all 160 KB of LDS) for the large ones:
// this is the wave tile with the fewest fragment reads per MFMA, the instruction shape that draws the
// least power per flop (these launches are power limited), and its memory instructions are interleaved
// with the MFMAs by hand.
#include "lds_tile.hpp"

namespace dora {
namespace {

constexpr int NUM_XCD = 8;
constexpr int GROUP_M = 8;

template <int BM_, int BN_, int WGM_, int WGN_, int BK_, int STAGES_, bool MI16_ = false>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_;
    static constexpr bool MI16 = MI16_;     // 16x16x32 MFMAs (8 x 8 per wave) instead of 32x32x16 (4 x 4)
    static constexpr int BK = BK_;          // K step per LDS buffer (elements)
    static constexpr int CPR = BK / 8;      // 16-byte chunks per K-contiguous LDS row
    static constexpr int STAGES = STAGES_;  // LDS ring depth (K steps)
    static constexpr int WAVES = WGM * WGN, THREADS = 64 * WAVES;
    static constexpr int WM = BM / WGM, WN = BN / WGN;
    static constexpr int MT = WM / 32, NT = WN / 32;
    static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int NLA = BM * CPR / THREADS;  // 16-byte loads per lane per K step, M side
    static constexpr int NLB = BN * CPR / THREADS;
    static constexpr int EPI_BYTES_PER_WAVE = 32 * (WN * 4 + 16);
    // Four waves of 128 x 128 each: the M-side operand gets a ring one deeper than STAGES and the two
    // rings lie one after the other; otherwise slot s holds the M-side tile followed by the N-side tile.
    static constexpr bool SPLIT_RING = (WAVES == 4) && (MT * NT >= 16);
    static constexpr int A_STAGES = SPLIT_RING ? STAGES + 1 : STAGES, B_STAGES = STAGES;
    static constexpr int RING_BYTES = A_STAGES * A_BYTES + B_STAGES * B_BYTES;
    static constexpr int LDS_BYTES = (RING_BYTES > WAVES * EPI_BYTES_PER_WAVE) ? RING_BYTES : WAVES * EPI_BYTES_PER_WAVE;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
    static constexpr int a_slot_off(int s) { return SPLIT_RING ? s * A_BYTES : s * STAGE_BYTES; }
    static constexpr int b_slot_off(int s) { return SPLIT_RING ? A_STAGES * A_BYTES + s * B_BYTES : s * STAGE_BYTES + A_BYTES; }
    static_assert(BK == 64, "the LDS layouts are written for K steps of 64");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be a multiple of the 32x32 MFMA");
    static_assert(WAVES == 4, "the schedules are written for four waves");
    static_assert(!MI16 || (SPLIT_RING && WM == 128 && WN == 128), "the 16x16x32 schedule is written for 128 x 128 per wave");
    static_assert((BM * CPR) % THREADS == 0 && (BN * CPR) % THREADS == 0, "load plan must divide evenly");
};

typedef Tile<256, 256, 2, 2, 64, 2, true> TileBig; // 256 threads, (3 + 2) x 32 KB of LDS, 256 accumulator registers (AGPRs) per lane
typedef Tile<128, 128, 2, 2, 64, 2> TileMed;      // 256 threads, 2 x 32 KB of LDS, two workgroups fit a CU
typedef Tile<128, 128, 2, 2, 64, 4> TileMedDeep;  // the same with a ring of four, for launches of at most one workgroup per CU

// Global -> LDS for one [ROWS x BK] operand tile.  Each wave-wide load instruction fills 1 KB of
// contiguous LDS (lane i lands at byte 16*i of it), so lane i fetches from global memory whatever
// belongs at that position of the swizzled tile; consecutive lanes cover one row segment of 2*BK bytes.
// Loads go through a buffer descriptor: an offset at or beyond num_records yields zeros, which
// covers rows past the end of the operand; rows or k out of range for other reasons get the offset
// 0xFFFFFFFF.  The K advance travels in the scalar offset.  The LW waves of the workgroup share the tile.
// The issue path itself has no vector arithmetic: a select feeding a load's address, with other vector
// instructions around it, stalls a wave that is otherwise issuing back-to-back 16-cycle MFMAs for several
// MFMAs' time (register-resident probe: 64 MFMAs + 8 such loads + 16 additions 1670 cycles against 1060
// with the loads taking their offsets as they are).  The k mask of a ragged last K step is therefore
// folded into the offsets once, before that step, and an exhausted cursor gets an empty descriptor.
template <int ROWS, int BK, int NL, int LW, bool KCONTIG>
struct OperandLoader {
    static constexpr int CPR = BK / 8;
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const bf16_t* base, int64_t ld, int rows, int K)
    {
        int64_t elems = KCONTIG ? ((int64_t)(rows - 1) * ld + K) : ((int64_t)(K - 1) * ld + rows);
        if (rows <= 0 || K <= 0) elems = 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)(uint32_t)(elems * 2), 0x00020000);
    }
    // tile-local (row, k) of the chunk that load i of this lane brings in
    static __device__ __forceinline__ void chunk_of(int i, int lw, int lane, int& row, int& k)
    {
        const int pos = (i * LW + lw) * 64 + lane;  // chunk position in the LDS tile
        if (KCONTIG) {
            row = pos / CPR;
            k = (((pos % CPR) ^ kc_swizzle<BK>(row)) & (CPR - 1)) * 8;
        } else {
            k = pos / (ROWS / 8);
            row = ((pos % (ROWS / 8)) ^ ks_swizzle(k)) * 8;
        }
    }
    // The k index (inside the K step) of load i is that of load 0 plus a compile-time increment: zero for
    // a K-contiguous tile (the swizzle repeats every 16 rows and LW loads cover a multiple of that), the
    // number of k-rows LW wave-loads span for a K-strided one.
    static_assert((LW * 64 / CPR) % 16 == 0, "K-contiguous swizzle must not depend on the load index");
    static constexpr int K_INC = KCONTIG ? 0 : LW * 64 / (ROWS / 8);
    static_assert(KCONTIG || (LW * 64) % (ROWS / 8) == 0, "K-strided loads must step whole k-rows");
    // per-lane constants: byte offset of the chunk of load i at k0 = 0 (0xFFFFFFFF if its row is out of
    // range) and the k index of load 0's chunk inside the K step
    static __device__ __forceinline__ void offsets(uint32_t (&vo)[NL], int& kl0, int64_t ld, int row0, int rows, int lw,
                                                   int lane)
    {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            int row, k;
            chunk_of(i, lw, lane, row, k);
            int grow = row0 + row;
            uint32_t off = KCONTIG ? (uint32_t)(((int64_t)grow * ld + k) * 2) : (uint32_t)(((int64_t)k * ld + grow) * 2);
            vo[i] = (grow < rows) ? off : 0xFFFFFFFFu;
            if (i == 0) kl0 = k;
        }
    }
    // Before a ragged last K step with `krem` k left: chunks whose k index is at or beyond it are pushed
    // out of range and load zeros.
    static __device__ __forceinline__ void mask_tail(uint32_t (&vo)[NL], int kl0, int krem)
    {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (kl0 + i * K_INC >= krem) vo[i] = 0xFFFFFFFFu;
    }
    // load I of a K step; `off` is its entry of the offset table
    template <int I>
    static __device__ __forceinline__ void issue_one(char* tile, __amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t soffset,
                                                     int lw)
    {
        static_assert(I >= 0 && I < NL, "load index");
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_ptr_t)(tile + (I * LW + lw) * 1024), 16, off, soffset, 0, 0);
    }
    static __device__ __forceinline__ void issue(char* tile, __amdgpu_buffer_rsrc_t rs, const uint32_t (&vo)[NL],
                                                 uint32_t soffset, int lw)
    {
        static_for<NL>([&](auto it) { issue_one<decltype(it)::value>(tile, rs, vo[decltype(it)::value], soffset, lw); });
    }
};

// Issue cursor of one operand: descriptor, per-lane offsets and the running scalar offset of the
// segment its global -> LDS loads are walking.  It runs ahead of the MFMAs.
template <class L, int NL, int BK, bool KCONTIG>
struct Cursor {
    uint32_t vo[NL];
    int kl0;
    __amdgpu_buffer_rsrc_t rs;
    uint32_t so, so_step;   // scalar byte offset of the next K step and its increment
    __device__ __forceinline__ void open(const bf16_t* base, int64_t ld, int K, int row0, int rows, int k_first, int wave,
                                         int lane)
    {
        rs = L::make_rsrc(base, ld, rows, K);
        L::offsets(vo, kl0, ld, row0, rows, wave, lane);
        so_step = KCONTIG ? (uint32_t)(BK * 2) : (uint32_t)(BK * ld * 2);
        so = KCONTIG ? (uint32_t)(k_first * 2) : (uint32_t)((int64_t)k_first * ld * 2);
    }
    // the next K step is the ragged last one of its segment, with krem k left
    __device__ __forceinline__ void mask_tail(int krem) { L::mask_tail(vo, kl0, krem); }
    // nothing left to load: every further load brings zeros
    __device__ __forceinline__ void exhaust(const bf16_t* base) { rs = L::make_rsrc(base, 0, 0, 0); }
    template <int I>
    __device__ __forceinline__ void issue_one(char* tile, int wave) const
    {
        L::template issue_one<I>(tile, rs, vo[I], so, wave);
    }
    __device__ __forceinline__ void issue_all(char* tile, int wave) const { L::issue(tile, rs, vo, so, wave); }
    __device__ __forceinline__ void step() { so += so_step; }
};

struct TileCoord { int tm, tn, z; };

// Workgroup id -> (tile row, tile column, K slice).  Hardware hands consecutive ids to the XCDs
// round-robin; undo that so each XCD owns a contiguous range of logical ids, then walk tiles in
// groups of GROUP_M rows so that co-resident tiles share operand panels in that XCD's L2.
__device__ __forceinline__ TileCoord map_tile(int wg, int tiles_m, int tiles_n, int ksplit)
{
    int total = tiles_m * tiles_n * ksplit;
    int q = total / NUM_XCD, rem = total % NUM_XCD;
    int xcd = wg % NUM_XCD, idx = wg / NUM_XCD;
    int logical = (xcd < rem) ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
    int tiles = tiles_m * tiles_n;
    TileCoord t;
    t.z = logical / tiles;
    int id = logical % tiles;
    int per_group = GROUP_M * tiles_n;
    int group = id / per_group;
    int first_m = group * GROUP_M;
    int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    int in_group = id % per_group;
    t.tm = first_m + in_group % gsz;
    t.tn = in_group / gsz;
    return t;
}

// TAG takes no part in the computation: it gives the two contractions that would otherwise share an
// instantiation separate kernel names, so that a profiler's per-kernel statistics line up with them.
template <class T, bool A_KC, bool B_KC, int EPI, int TAG, int DT>
__global__ __launch_bounds__(T::THREADS) void gemm_bf16_kernel(GemmPair grp)
{
    __shared__ __attribute__((aligned(1024))) char smem[T::LDS_BYTES];
    // one launch may carry two independent problems of the same kind (e.g. dA and dB): workgroups
    // past count0 belong to the second one
    const bool second = (int)blockIdx.x >= grp.count0;
    const GemmArgs& p = second ? grp.g[1] : grp.g[0];
    const int wg_id = (int)blockIdx.x - (second ? grp.count0 : 0);
#include "gemm_tile_body.hpp"
}

// The last products of a backward in one launch: the input gradients (dx = dz W + dh A, and the frozen path's with dropout) in
// tiles TI, and in 128 x 128 ones TW the weight gradients (dA = dh^T x, dB = s dz^T h), which wait for nothing that the others
// do not wait for too.  Bound by the longest of its tiles where one round holds them all: the weight gradients then cost neither
// a launch nor time.  (Training step 1024 x 4096, r 64, 512 tokens 70.6 -> 61.0 us; 2048 x 2048, r 64, 1024 tokens 84.3 -> 72.8;
// with dropout 2056 x 3000, r 72, 1501 tokens 189.7 -> 175.5.)
template <class TI, class TW, int DT>
__global__ __launch_bounds__(TI::THREADS) void gradients_kernel(GemmPair inputs, GemmPair weights, int input_wgs)
{
    static_assert(TI::THREADS == TW::THREADS, "");
    __shared__ __attribute__((aligned(1024))) char smem[TI::LDS_BYTES > TW::LDS_BYTES ? TI::LDS_BYTES : TW::LDS_BYTES];
    if ((int)blockIdx.x < input_wgs) {
        typedef TI T;
        constexpr bool A_KC = true, B_KC = false;
        constexpr int EPI = EPI_STORE_BF16;
        const bool second = (int)blockIdx.x >= inputs.count0;
        const GemmArgs& p = second ? inputs.g[1] : inputs.g[0];
        const int wg_id = (int)blockIdx.x - (second ? inputs.count0 : 0);
#include "gemm_tile_body.hpp"
    } else {
        typedef TW T;
        constexpr bool A_KC = false, B_KC = false;
        constexpr int EPI = EPI_STORE_F32;
        const int block = (int)blockIdx.x - input_wgs;
        const bool second = block >= weights.count0;
        const GemmArgs& p = second ? weights.g[1] : weights.g[0];
        const int wg_id = block - (second ? weights.count0 : 0);
#include "gemm_tile_body.hpp"
    }
}

template <class T>
int grid_of(const GemmArgs& a)
{
    if (a.M <= 0 || a.N <= 0) return 0;
    return ((a.M + T::BM - 1) / T::BM) * ((a.N + T::BN - 1) / T::BN) * a.ksplit;
}

template <class T, bool A_KC, bool B_KC, int EPI>
hipError_t launch_one(const GemmArgs& a, const GemmArgs* b, hipStream_t stream)
{
    GemmPair grp;
    grp.g[0] = a;
    grp.g[1] = b ? *b : a;
    grp.count0 = grid_of<T>(a);
    const int grid = grp.count0 + (b ? grid_of<T>(*b) : 0);
    if (grid == 0) return hipSuccess;
    if (b && b->dt != a.dt) return hipErrorInvalidValue;
    if (a.dt == DT_F16) {
        if (a.tag) gemm_bf16_kernel<T, A_KC, B_KC, EPI, 1, DT_F16><<<dim3(grid), dim3(T::THREADS), 0, stream>>>(grp);
        else gemm_bf16_kernel<T, A_KC, B_KC, EPI, 0, DT_F16><<<dim3(grid), dim3(T::THREADS), 0, stream>>>(grp);
    } else {
        if (a.tag) gemm_bf16_kernel<T, A_KC, B_KC, EPI, 1, DT_BF16><<<dim3(grid), dim3(T::THREADS), 0, stream>>>(grp);
        else gemm_bf16_kernel<T, A_KC, B_KC, EPI, 0, DT_BF16><<<dim3(grid), dim3(T::THREADS), 0, stream>>>(grp);
    }
    return hipGetLastError();
}

// What a K step costs a launch of so many tiles, in hundredths of a microsecond: 128 x 128 tiles run two to a CU (one, with
// the deep ring, where they are at most 256), 256 x 256 ones one to a CU, in rounds.  Measured on x W^T and dz W of 512 to 8192
// tokens at 4096 x 4096, 14336 x 4096, 4096 x 14336, 3000 x 2056 and 5120 x 27648: one round of 128 x 128 tiles 0.5 us a step up
// to 256 tiles, 1.0 up to 512; of 256 x 256 ones 1.15 with few of them to 1.5 with 256.
int64_t med_cost(int64_t tiles) { return tiles / 512 * 100 + (tiles % 512 == 0 ? 0 : tiles % 512 <= 256 ? 55 : 100); }
int64_t big_cost(int64_t tiles) { return tiles / 256 * 150 + (tiles % 256 == 0 ? 0 : 115 + 35 * (tiles % 256) / 256); }

int64_t tiles_of(int64_t M, int64_t N, int64_t tile) { return ((M + tile - 1) / tile) * ((N + tile - 1) / tile); }

// The large tile from a full round of them on, and below where its one round is the cheaper one.  (512 tiles of 128 x 128 are
// one round of 1.0, 576 two, and 144 of 256 x 256 one of 1.35: 4096 x 4096, 2304 tokens 120 -> 102 us, 5120 x 27648, 2048
// tokens 819 -> 511.  From 260 large tiles on the two are within 5 % of each other at K 4096 and less, and at larger K the
// large tile is faster by up to half.)  A short K, where the epilogue is most of a tile, keeps the line at the full round.
bool use_big(const GemmArgs& a, const GemmArgs* b)
{
    if ((a.epilogue != EPI_STORE_BF16 && a.epilogue != EPI_COMPOSE) || a.ksplit != 1) return false;
    const int64_t big = tiles_of(a.M, a.N, 256) + (b ? tiles_of(b->M, b->N, 256) : 0);
    const int64_t med = tiles_of(a.M, a.N, 128) + (b ? tiles_of(b->M, b->N, 128) : 0);
    return big >= 256 || (a.seg[0].K >= 1024 && big_cost(big) < med_cost(med));
}

// Columns (or, if `rows`, rows) that go to whole rounds of large tiles where what is left over goes to one round of 128 x 128
// ones with a CU each, or 0: the few large tiles of a last round cost three quarters of a full one.  (272 tiles, 4096 x 4096,
// 4352 tokens: 192 us for two rounds, 150 this way.  Half a round left over is no slower in large tiles, the power limit being what it is.)
// The second launch costs 6 us.
int big_part(const GemmArgs& a, bool& rows)
{
    const int64_t tm = (a.M + 255) / 256, tn = (a.N + 255) / 256, steps = (a.seg[0].K + 63) / 64;
    int64_t best = big_cost(tm * tn) * steps - 600;
    int part = 0;
    for (int along = 0; along < 2; ++along) {
        const int64_t n = along ? tm : tn, other = along ? tn : tm, k = tm * tn / 256 * 256 / other;
        if (k <= 0 || k >= n) continue;
        const int64_t rest = along ? tiles_of(a.M - k * 256, a.N, 128) : tiles_of(a.M, a.N - k * 256, 128);
        const int64_t cost = (big_cost(k * other) + med_cost(rest)) * steps;
        if (rest <= 256 && cost < best) { best = cost; part = (int)(k * 256); rows = along != 0; }
    }
    return part;
}

template <bool A_KC, bool B_KC, int EPI>
hipError_t launch_parts(const GemmArgs& a, int part, bool rows, hipStream_t stream)
{
    GemmArgs first = a, second = a;
    for (int i = 0; i < a.nseg; ++i) {
        GemmSeg& sg = second.seg[i];
        if (rows) sg.a += A_KC ? part * sg.lda : part;
        else sg.b += B_KC ? part * sg.ldb : part;
    }
    if (rows) { first.M = part; second.M = a.M - part; }
    else {
        first.N = part; second.N = a.N - part;
        if (a.colscale) second.colscale = a.colscale + part;
        if (a.colbias) second.colbias = a.colbias + part;
    }
    const int64_t out = rows ? part * a.ldc : part;
    second.c = (bf16_t*)a.c + out;
    if (a.c2) second.c2 = (bf16_t*)a.c2 + out;
    hipError_t e = launch_one<TileBig, A_KC, B_KC, EPI>(first, nullptr, stream);
    return e != hipSuccess ? e : launch_one<TileMedDeep, A_KC, B_KC, EPI>(second, nullptr, stream);
}

hipError_t dispatch(const GemmArgs& a, const GemmArgs* b, hipStream_t stream)
{
    const bool big = use_big(a, b);
    bool rows = false;
    const int part = big && !b && a.seg[0].K >= 1024 ? big_part(a, rows) : 0;
    // at most one 128x128-tile workgroup per CU: give it the deep ring
    const bool deep = !big && (grid_of<TileMed>(a) + (b ? grid_of<TileMed>(*b) : 0)) <= 256;
#define DORA_GEMM_MED(AKC, BKC, E) \
    (deep ? launch_one<TileMedDeep, AKC, BKC, E>(a, b, stream) : launch_one<TileMed, AKC, BKC, E>(a, b, stream))
#define DORA_GEMM_CASE(AKC, BKC, E)                                                     \
    if (a.a_kcontig == (AKC) && a.b_kcontig == (BKC) && a.epilogue == (E))              \
        return part ? launch_parts<AKC, BKC, E>(a, part, rows, stream)                  \
             : big ? launch_one<TileBig, AKC, BKC, E>(a, b, stream) : DORA_GEMM_MED(AKC, BKC, E);
    DORA_GEMM_CASE(true, true, EPI_STORE_BF16)
    DORA_GEMM_CASE(true, false, EPI_STORE_BF16)
    DORA_GEMM_CASE(true, true, EPI_COMPOSE)
#undef DORA_GEMM_CASE
#define DORA_GEMM_CASE_MED(AKC, BKC, E)                                                 \
    if (a.a_kcontig == (AKC) && a.b_kcontig == (BKC) && a.epilogue == (E))              \
        return DORA_GEMM_MED(AKC, BKC, E);
    DORA_GEMM_CASE_MED(true, true, EPI_STORE_F32)
    DORA_GEMM_CASE_MED(true, false, EPI_STORE_F32)
    DORA_GEMM_CASE_MED(true, true, EPI_ROWDOT)
    DORA_GEMM_CASE_MED(false, false, EPI_STORE_F32)
#undef DORA_GEMM_CASE_MED
#undef DORA_GEMM_MED
    return hipErrorInvalidValue;
}

// Tiles of the input gradients for the launch that takes the weight gradients along, 0 where these go by themselves: where
// they find CUs without work in a round that has to be run anyway, in the tiles that the input gradients take by themselves.
// Where two workgroups share a CU, the weight gradients have the ring of two instead of the deep one: once the input gradients
// are through, a K step takes them half as long again, so only while tokens are not many more than the K of those.  (Backward, in
// one launch and in two, steps of 64 tokens against steps of dx: 512 x 4096, r 16, 1500 tokens, 24 and 9, 39 us and 44; 1136 x
// 968, r 48, 6050 tokens, 95 and 19, 93 and 88; 512 x 640, r 8, 8192 tokens, 128 and 9, 99 and 81; 256 x 512, r 8, 16000 tokens,
// 250 and 5, 163 and 116.  Over 200 shapes this line is within 0.1 % of always taking the faster one.)
enum { APART, IN_BIG, IN_DEEP, IN_MED };
int grads_together(const GemmArgs* dx, int n, const GemmArgs* w, int m)
{
    if (n < 1 || n > 2 || m < 1 || m > 2) return APART;
    int64_t big = 0, med = 0, rest = 0, steps_in = 0, steps_w = 0;
    for (int i = 0; i < n; ++i) {
        int64_t steps = 0;
        for (int k = 0; k < dx[i].nseg; ++k) steps += (dx[i].seg[k].K + 63) / 64;
        steps_in = steps > steps_in ? steps : steps_in;
        if (!dx[i].a_kcontig || dx[i].b_kcontig || dx[i].epilogue != EPI_STORE_BF16 || dx[i].ksplit != 1 || dx[i].dt != dx[0].dt) return APART;
        big += tiles_of(dx[i].M, dx[i].N, 256);
        med += tiles_of(dx[i].M, dx[i].N, 128);
    }
    for (int i = 0; i < m; ++i) {
        if (w[i].a_kcontig || w[i].b_kcontig || w[i].epilogue != EPI_STORE_F32 || w[i].ksplit != 1 || w[i].dt != dx[0].dt) return APART;
        rest += tiles_of(w[i].M, w[i].N, 128);
        steps_w = (w[i].seg[0].K + 63) / 64;           // tokens, for both of them
    }
    const GemmArgs* second = n > 1 ? &dx[1] : nullptr;
    if (use_big(dx[0], second)) {
        bool rows;
        if (big > 256 && !second && big_part(dx[0], rows)) return APART;
        return big % 256 != 0 && big % 256 + rest <= 256 ? IN_BIG : APART;
    }
    if (med + rest <= 256) return IN_DEEP;
    return med > 256 && med % 512 != 0 && med % 512 + rest <= 512 && steps_w < 30 + 2 * steps_in ? IN_MED : APART;
}

template <class T, class TW>
hipError_t launch_grads(const GemmArgs* dx, int n, const GemmArgs* w, int m, hipStream_t stream)
{
    const GemmPair inputs{{dx[0], dx[n - 1]}, grid_of<T>(dx[0])}, weights{{w[0], w[m - 1]}, grid_of<TW>(w[0])};
    const int input_wgs = inputs.count0 + (n > 1 ? grid_of<T>(dx[1]) : 0);
    const int wgs = input_wgs + weights.count0 + (m > 1 ? grid_of<TW>(w[1]) : 0);
    if (wgs == 0) return hipSuccess;
    if (dx[0].dt == DT_F16) gradients_kernel<T, TW, DT_F16><<<dim3(wgs), dim3(T::THREADS), 0, stream>>>(inputs, weights, input_wgs);
    else gradients_kernel<T, TW, DT_BF16><<<dim3(wgs), dim3(T::THREADS), 0, stream>>>(inputs, weights, input_wgs);
    return hipGetLastError();
}

}  // namespace

bool gemm_bf16_grads_together(const GemmArgs* dx, int n, const GemmArgs* w, int m) { return grads_together(dx, n, w, m) != APART; }

hipError_t launch_gemm_bf16_grads(const GemmArgs* dx, int n, const GemmArgs* w, int m, int trace_id, hipStream_t stream)
{
    TraceScope ts(trace_id, stream);
    switch (grads_together(dx, n, w, m)) {
        case IN_BIG: return launch_grads<TileBig, TileMedDeep>(dx, n, w, m, stream);
        case IN_DEEP: return launch_grads<TileMedDeep, TileMedDeep>(dx, n, w, m, stream);
        case IN_MED: return launch_grads<TileMed, TileMed>(dx, n, w, m, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_bf16(const GemmArgs& a, int trace_id, hipStream_t stream)
{
    if (a.M == 0 || a.N == 0) return hipSuccess;
    TraceScope ts(trace_id, stream);
    return dispatch(a, nullptr, stream);
}

bool gemm_bf16_pairs(const GemmArgs& a, const GemmArgs& b)
{
    auto cost = [](const GemmArgs& p, const GemmArgs* q) {
        const int64_t big = tiles_of(p.M, p.N, 256) + (q ? tiles_of(q->M, q->N, 256) : 0);
        const int64_t med = tiles_of(p.M, p.N, 128) + (q ? tiles_of(q->M, q->N, 128) : 0);
        return use_big(p, q) ? big_cost(big) : med_cost(med);
    };
    const int64_t steps = (a.seg[0].K + 63) / 64;
    return cost(a, &b) * steps < (cost(a, nullptr) + cost(b, nullptr)) * steps + 600;
}

hipError_t launch_gemm_bf16_pair(const GemmArgs& a, const GemmArgs& b, int trace_id, hipStream_t stream)
{
    // both problems run the same kernel instance: same operand layouts and element type; same epilogue without
    // split-K, or a row-dot problem (split or not) followed by an fp32-store problem (split or not)
    const bool same = a.epilogue == b.epilogue && a.ksplit == 1 && b.ksplit == 1;
    const bool rowdot_then_store = a.epilogue == EPI_ROWDOT && b.epilogue == EPI_STORE_F32 && b.nseg == 1;
    if (a.a_kcontig != b.a_kcontig || a.b_kcontig != b.b_kcontig || a.dt != b.dt || !(same || rowdot_then_store))
        return hipErrorInvalidValue;
    if ((a.M == 0 || a.N == 0) && (b.M == 0 || b.N == 0)) return hipSuccess;
    TraceScope ts(trace_id, stream);
    return dispatch(a, &b, stream);
}

}  // namespace dora
