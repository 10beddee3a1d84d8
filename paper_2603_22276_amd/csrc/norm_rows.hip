// The three sums of the row norm (Eq. 2) in one launch, 16-bit storage, ranks up to NORM_ROWS_MAX_RANK:
//
//   base[m] = sum_n W[m,n]^2,   cross[m] = sum_n W[m,n] V[m,n],   ba[m] = sum_n V[m,n]^2,   V = B A
//
// V lives in the accumulators of one 128 x 128 tile at a time and is never stored.  Its products are as many as those of
// U = W A^T (2 d_out d_in r), but W meets V element by element, so the Gram matrix, B G and the launches between them are not
// needed for the norm, and both low-rank sums come from fp32 values.
//
// Bound: reading W once up to r about 128, the matrix cores beyond.  A workgroup of four waves, 2 x 2 over a tile, keeps 128
// rows of B in registers as MFMA fragments (r / 2 of them per lane) and walks over column tiles: the K steps of A, 64 x 128
// each, and the tile of W in two halves go through one ring of 16 KB LDS slots filled by direct loads, so the loads of the
// next tiles are in flight whatever is being multiplied.  With B out of the LDS a K step costs it 32 KB of fragment reads and
// 16 KB of loads for 512 cycles of MFMA; with both operands in it, as in the 128 x 128 tile of the other products, 64 and
// 32 KB, which is what bounds that tile.
//
// Against four launches (W A^T with its row sums and A A^T, the sum of the slices of G, B G, Eq. 5), repeated calls over one W,
// us of a norm with Eq. 5: 8192 x 8192, r 128 46 -> 35 (29 of it this launch, 4.6 TB/s), r 384 83 -> 58; 4096 x 4096, r 384
// 43 -> 23; 14336 x 4096, r 384 93 -> 59; 27648 x 5120, r 384 179 -> 133; 1024 x 4096, r 64 24 -> 11.  104 shapes 1.15 to 3
// times faster; the error against 64 bits 5.5e-8 -> 5.0e-8 on average (largest 7.7e-8 -> 5.5e-8).
#include "lds_tile.hpp"

namespace dora {
namespace {

constexpr int BM = 128, BN = 128;
constexpr int SLOT = 16384;                            // 64 k x 128 columns of A, or 2 x 32 rows x 128 columns of W
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
constexpr uint32_t OUTSIDE = 0xFFFFFFFFu;              // beyond every descriptor: loads zeros

// 8 bytes of LDS per lane, left as one value until its wait: taking it apart is an instruction
template <int OFF>
__device__ __forceinline__ uint64_t lds_read_b64(uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "ds_read offset field is 16 bits");
    uint64_t v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}

// Where a workgroup stands, and its loads.
template <int S>   // K steps of 64 that hold r
struct Walk {
    static constexpr int LPS = 4;                      // wave-wide loads of 1 KB per slot and wave
    static constexpr int PER_TILE = S + 2;             // slots of a tile: K steps of A, then W in two halves
    int slice, m0, rows, t_begin, t_end, d_in, wave;
    uint32_t ld;
    __amdgpu_buffer_rsrc_t ra, rw;
    uint32_t va, val[LPS], vw[2][LPS];
    int acol, wcol[2];

    __device__ __forceinline__ Walk(const NormRowsArgs& p, int wave_, int lane) : d_in(p.d_in), wave(wave_)
    {
        // consecutive ids go to the XCDs in turn: undone, so that an XCD (own L2) works on all slices of its row blocks and
        // reads their rows of B once
        const int total = (p.d_out + BM - 1) / BM * p.slices;
        const int wg = blockIdx.x, xcd = wg & 7, xq = total >> 3, xr = total & 7;
        const int logical = (xcd < xr ? xcd * (xq + 1) : xr * (xq + 1) + (xcd - xr) * xq) + (wg >> 3);
        slice = logical % p.slices;
        m0 = logical / p.slices * BM;
        rows = p.d_out - m0 < BM ? p.d_out - m0 : BM;
        const int tiles = (d_in + BN - 1) / BN;
        t_begin = slice * p.tiles_per_slice;
        t_end = t_begin + p.tiles_per_slice < tiles ? t_begin + p.tiles_per_slice : tiles;

        // The row and column of a lane travel in the vector offset, which alone is range checked; what is the same for all
        // lanes (K step, column tile, row of a load) in the scalar one.
        ld = (uint32_t)d_in * 2u;
        ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.a), 0, (int)(uint32_t)((int64_t)p.r * d_in * 2), 0x00020000);
        rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.w + (int64_t)m0 * d_in), 0,
                                               (int)(uint32_t)((int64_t)rows * d_in * 2), 0x00020000);
        // A: load i of a wave brings k = 16 i + 4 wave + lane / 16 of a K step; its column does not depend on i.  `val`: the
        // last K step, whose k may lie past r.
        const int ak = wave * 4 + (lane >> 4);
        acol = ((lane & 15) ^ ks_swizzle(ak)) * 8;
        va = (uint32_t)ak * ld + (uint32_t)acol * 2u;
#pragma unroll
        for (int i = 0; i < LPS; ++i) val[i] = (S - 1) * 64 + i * 16 + ak < p.r ? va : OUTSIDE;
        // W: load i of half h brings rows 32 h + 8 i + lane / 8 of the wave's own 64, in chunks swizzled by row / 2
        const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
#pragma unroll
        for (int i = 0; i < LPS; ++i) {
            if (i < 2) wcol[i] = wn0 + ((lane & 7) ^ ((i * 4 + (lane >> 4)) & 7)) * 8;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = wm0 + h * 32 + i * 8 + (lane >> 3);
                vw[h][i] = row < rows ? (uint32_t)(wm0 + (lane >> 3)) * ld + (uint32_t)wcol[i & 1] * 2u : OUTSIDE;
            }
        }
    }
    // The loads take their offsets as they are.  Column tiles come in ascending order, so what lies past the end of W's and
    // A's columns, or past the slice, is masked for good before the first load of the tile where it begins.
    __device__ __forceinline__ void open_tile(int t)
    {
        const int cols = t < t_end ? d_in - t * BN : 0;
        if (cols >= BN) return;
        if (acol >= cols) {
            va = OUTSIDE;
#pragma unroll
            for (int i = 0; i < LPS; ++i) val[i] = OUTSIDE;
        }
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            if (wcol[i & 1] >= cols) vw[0][i] = vw[1][i] = OUTSIDE;
    }
    // load I of slot SEQ of the walk, counted from the first of tile t
    template <int SEQ, int I>
    __device__ __forceinline__ void issue_one(int t, char* slot)
    {
        constexpr int K = SEQ % PER_TILE;              // K step of A, or S + half of W
        t += SEQ / PER_TILE;
        if constexpr (K == 0 && I == 0) open_tile(t);
        const uint32_t so = (uint32_t)t * (BN * 2u);
        if constexpr (K < S)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_ptr_t)(slot + (I * 4 + wave) * 1024), 16, K == S - 1 ? val[I] : va,
                                                     so + (K * 64 + I * 16) * ld, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void_ptr_t)(slot + wave * 4096 + I * 1024), 16, vw[K - S][I],
                                                     so + ((K - S) * 32 + I * 8) * ld, 0, 0);
    }
    template <int SEQ>
    __device__ __forceinline__ void issue(int t, char* slot)
    {
        static_for<LPS>([&](auto it) { issue_one<SEQ, decltype(it)::value>(t, slot); });
    }
};

// LDS reads of a lane, relative to the slot: fragments of A's column block j, W's values against it
__device__ __forceinline__ void read_offsets(uint32_t smem_lds, int wave, int lane, uint32_t (&rb)[4], uint32_t (&rw)[4])
{
    const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        rb[j] = smem_lds + frag16_off<BN, 64, false>((wave & 1) * 64 + j * 16, 0, lane);
        rw[j] = smem_lds + (uint32_t)(wave * 4096 + l16 * 128 + (((2 * j + (lq >> 1)) ^ (l16 >> 1)) & 7) * 16 + (lq & 1) * 8);
    }
}

// a workgroup's sums leave: over the four lanes and two waves that share a row
__device__ __forceinline__ void store_sums(const NormRowsArgs& p, float* red, const float (&sum)[3][4], int wave, int lane, int slice,
                                           int m0, int rows)
{
    __syncthreads();                                   // red: [2 halves of the columns][3][BM]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float v = sum[k][i];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (lane < 16) red[((wave & 1) * 3 + k) * BM + (wave >> 1) * 64 + i * 16 + lane] = v;
        }
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * BM; e += 256) {
        const int k = e / BM, m = e % BM;
        if (m < rows) p.part[((int64_t)k * p.slices + slice) * p.d_out + m0 + m] = red[e] + red[3 * BM + e];
    }
}

typedef __attribute__((address_space(3))) const char* lds_cptr_t;

// Ranks up to 128: two workgroups to a CU, one's sums beside the other's products (8192 x 8192, r 128 29 us against 33 for the
// kernel below).
template <int S, int DT>
__global__ __launch_bounds__(256, 2) void norm_rows_kernel(NormRowsArgs p)
{
    typedef Elem16<DT> E;
    typedef Walk<S> Wk;
    constexpr int NS = 5, LPS = Wk::LPS, PER_TILE = Wk::PER_TILE;
    __shared__ __attribute__((aligned(1024))) char smem[NS * SLOT];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    Wk walk(p, wave, lane);

    // B as fragments: lane (l16, lq) of block i, k-step q of 32 holds row 16 i + l16, k = 32 q + 8 lq .. +7
    bf16x8_t bf[2 * S][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (wave >> 1) * 64 + i * 16 + l16;
        const bf16_t* const src = p.b + (int64_t)(walk.m0 + (row < walk.rows ? row : walk.rows - 1)) * p.r;
#pragma unroll
        for (int q = 0; q < 2 * S; ++q) {
            const int k = q * 32 + lq * 8;
            uint4 v = *reinterpret_cast<const uint4*>(src + (k < p.r ? k : 0));
            if (k >= p.r) v = make_uint4(0u, 0u, 0u, 0u);
            bf[q][i] = __builtin_bit_cast(bf16x8_t, v);
        }
    }
    static_for<NS - 1>([&](auto nt) { walk.template issue<decltype(nt)::value>(walk.t_begin, smem + decltype(nt)::value * SLOT); });
#pragma unroll
    for (int q = 0; q < 2 * S; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(bf[q][i]));   // landed, and in registers from here on

    uint32_t rb[4], rwd[4];
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(lds_cptr_t)smem;
    read_offsets(smem_lds, wave, lane, rb, rwd);
    float sum[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[k][i] = 0.f;
    int cur = 0;                                       // slot of the step under way; the one before it is refilled
    // the start of a step: its slot has landed and everyone is done with the one before
    auto enter = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt<(NS - 2) * LPS>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        return (uint32_t)cur * SLOT;
    };
    auto landed = [](bf16x8_t (&f)[4]) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = walk.t_begin; t < walk.t_end; ++t) {
        f32x4_t acc[4][4];
        bf16x8_t fx[4], fy[4];
        // the products of k-step q; step kind K >= 0: the loads of its refill behind every fourth
        auto mma = [&](auto q_tag, auto k_tag, const bf16x8_t (&f)[4]) {
            constexpr int q = decltype(q_tag)::value, K = decltype(k_tag)::value;
            static_for<16>([&](auto nt) {
                constexpr int n = decltype(nt)::value, i = n / 4, j = n % 4;
                acc[i][j] = E::mfma16(f[j], bf[q][i], q == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[i][j]);
                if constexpr (K >= 0 && j == 1) {
                    walk.template issue_one<K + NS - 1, i>(t, smem + (cur == 0 ? NS - 1 : cur - 1) * SLOT);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };
        static_for<S>([&](auto st) {
            constexpr int s = decltype(st)::value;
            const uint32_t slot = enter();
            static_for<4>([&](auto jt) { fx[decltype(jt)::value] = lds_read_tr<0, 4 * BN * 2>(slot + rb[decltype(jt)::value]); });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (s > 0) mma(std::integral_constant<int, 2 * s - 1>{}, st, fy);
            __builtin_amdgcn_sched_barrier(0);
            landed(fx);
            static_for<4>([&](auto jt) {
                fy[decltype(jt)::value] = lds_read_tr<32 * BN * 2, 4 * BN * 2>(slot + rb[decltype(jt)::value]);
            });
            __builtin_amdgcn_sched_barrier(0);
            mma(std::integral_constant<int, 2 * s>{}, std::integral_constant<int, s == 0 ? 0 : -1>{}, fx);
            __builtin_amdgcn_sched_barrier(0);
            landed(fy);
            cur = cur + 1 == NS ? 0 : cur + 1;
        });
        // W against the tile, 32 of a wave's 64 rows at a time
        static_for<2>([&](auto ht) {
            constexpr int h = decltype(ht)::value;
            const uint32_t slot = enter();
            uint64_t w[8];
            static_for<8>([&](auto nt) {
                constexpr int n = decltype(nt)::value;
                w[n] = lds_read_b64<n / 4 * 2048>(slot + rwd[n % 4]);
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (h == 0) mma(std::integral_constant<int, 2 * S - 1>{}, std::integral_constant<int, S>{}, fy);
            else walk.template issue<S + 1 + NS - 1>(t, smem + (cur == 0 ? NS - 1 : cur - 1) * SLOT);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int i = h * 2 + ii;
                // the sixteen products of a block first, then the running sum over tiles
                float tb = 0.f, tc = 0.f, ta = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u32x2_t w2 = __builtin_bit_cast(u32x2_t, w[ii * 4 + j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float wv = e % 2 ? E::hi(w2[e / 2]) : E::lo(w2[e / 2]), v = acc[i][j][e];
                        tb = fmaf(wv, wv, tb);
                        tc = fmaf(wv, v, tc);
                        ta = fmaf(v, v, ta);
                    }
                }
                sum[0][i] += tb; sum[1][i] += tc; sum[2][i] += ta;
            }
            cur = cur + 1 == NS ? 0 : cur + 1;
        });
    }
    wait_vmcnt<0>();                                   // the loads past the end have written their zeros
    store_sums(p, reinterpret_cast<float*>(smem), sum, wave, lane, walk.slice, walk.m0, walk.rows);
}

// 16 bytes of LDS per lane into accumulator registers, where MFMA operands that stay leave the others free
__device__ __forceinline__ bf16x8_t lds_read_b128_acc(uint32_t addr)
{
    bf16x8_t v;
    asm volatile("ds_read_b128 %0, %1" : "=a"(v) : "v"(addr));
    return v;
}

// Which load goes behind which MFMA of a tile.  A tile brings as many slots as it uses up, S + 2, and their loads are spread
// evenly, because a load that follows another too closely holds the wave up.  What it brings first goes where the last K step
// of the tile before was (everyone has read it at the first barrier, before MFMA 4), then where W of the tile before was and
// where its own K steps were (free at the barrier of the second K step, MFMA 36, and of the one after each).  `FIRST`
// slots are asked for before the first tile.
template <int S, int NS>
struct Refill {
    static constexpr int LPS = 4, LOADS = (S + 2) * LPS, MFMAS = 32 * S;
    static constexpr int FIRST = NS - 3;
    // the barrier from which on everyone has read what load l overwrites
    static constexpr int free_at(int l) { return l / LPS == 0 ? 4 : l / LPS <= 3 ? 36 : 36 + (l / LPS - 3) * 32; }
    // MFMA of the tile behind which load l of its refills goes
    static constexpr int place(int l)
    {
        int at = 16;
        for (int i = 1; i <= l; ++i) {
            const int gap = (MFMAS - at) / (LOADS - i + 1);
            at += gap > 1 ? gap : 1;
            if (at < free_at(i)) at = free_at(i);
        }
        return at;
    }
    // load behind MFMA m, as 4 * (slot of the walk, from the tile's first) + load, or -1
    static constexpr int load_at(int m)
    {
        for (int l = 0; l < LOADS; ++l)
            if (place(l) == m) return FIRST * LPS + l;
        return -1;
    }
    // loads asked for before MFMA m, from those of the tile's first slot on
    static constexpr int loads_before(int m)
    {
        int n = FIRST * LPS;
        for (int l = 0; l < LOADS; ++l) n += place(l) < m;
        return n;
    }
    static constexpr bool fits() { return place(LOADS - 1) < MFMAS; }
};

// Ranks past 128 (a wave's share of B does not leave room for a second wave on its SIMD): one workgroup to a CU, ten slots.  One wave per SIMD hides nothing by itself, so everything else is
// written between the MFMAs, about two instructions to each (what a 16-cycle MFMA takes for nothing; more of them cost five
// cycles each): the fragment reads, which are a whole half step ahead, the loads, and the sums of the tile before, whose
// accumulators move to vector registers as the first products of the next tile replace them.
template <int S, int DT>
__global__ __launch_bounds__(256, 1) void norm_rows_deep_kernel(NormRowsArgs p)
{
    typedef Elem16<DT> E;
    typedef Walk<S> Wk;
    constexpr int NS = 10, LPS = Wk::LPS;
    __shared__ __attribute__((aligned(1024))) char smem[NS * SLOT];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    Wk walk(p, wave, lane);
    const int r = p.r, rows = walk.rows;

    const uint32_t ldb = (uint32_t)r * 2u;
    const __amdgpu_buffer_rsrc_t rbs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.b + (int64_t)walk.m0 * r), 0,
                                                                         (int)(uint32_t)((int64_t)rows * r * 2), 0x00020000);
    // B, 64 k at a time into the last S slots: load i of a wave brings rows 32 i + 8 wave + lane / 8
    static_for<S * LPS>([&](auto nt) {
        constexpr int s = decltype(nt)::value / LPS, i = decltype(nt)::value % LPS;
        const int row = i * 32 + wave * 8 + (lane >> 3), k = s * 64 + ((lane & 7) ^ kc_swizzle<64>(row)) * 8;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rbs, (lds_void_ptr_t)(smem + (NS - S + s) * SLOT + (i * 4 + wave) * 1024), 16,
                                                 row < rows && k < r ? (uint32_t)row * ldb + (uint32_t)k * 2u : OUTSIDE, 0, 0, 0);
    });
    // Before the loop FIRST slots of the walk: beside B as many as there is room for, the others once B has left.
    static_assert(S >= 2 && Refill<S, NS>::fits(), "the loads of a tile");
    constexpr int FIRST = Refill<S, NS>::FIRST, BESIDE = FIRST < NS - S ? FIRST : NS - S;
    static_for<BESIDE>([&](auto nt) { walk.template issue<decltype(nt)::value>(walk.t_begin, smem + decltype(nt)::value * SLOT); });
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(lds_cptr_t)smem;
    wait_vmcnt<BESIDE * LPS>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // B as fragments: lane (l16, lq) of block i, k-step q of 32 holds row 16 i + l16, k = 32 q + 8 lq .. +7
    bf16x8_t bf[2 * S][4];
#pragma unroll
    for (int q = 0; q < 2 * S; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            bf[q][i] = lds_read_b128_acc(smem_lds + (NS - S + q / 2) * SLOT + (uint32_t)lds_off<64>((wave >> 1) * 64 + i * 16 + l16, q % 2 * 32 + lq * 8));
#pragma unroll
    for (int q = 0; q < 2 * S; ++q)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+a"(bf[q][0]), "+a"(bf[q][1]), "+a"(bf[q][2]), "+a"(bf[q][3]));
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    static_for<FIRST - BESIDE>([&](auto nt) {
        constexpr int n = BESIDE + decltype(nt)::value;
        walk.template issue<n>(walk.t_begin, smem + n * SLOT);
    });

    uint32_t rb[4], rwd[4];
    read_offsets(smem_lds, wave, lane, rb, rwd);
    float sum[3][4], part[3];                          // base, cross, ba of the four row blocks; of one block in one tile
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        part[k] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[k][i] = 0.f;
    }
    uint64_t w[4][4];
    f32x4_t old[4][4];
    // Instruction u of the sums over the products in `old` and W's in w: four to an element, whose order is row block, column
    // block, column.  The sixteen elements of a block first, then the running sum over tiles.
    float wv = 0.f;
    auto sums = [&](auto u_tag) {
        constexpr int u = decltype(u_tag)::value, e = u / 4, i = e / 16, j = e / 4 % 4, c = e % 4;
        const float v = old[i][j][c];
        if constexpr (u % 4 == 0) {
            const uint32_t w2 = __builtin_bit_cast(u32x2_t, w[i][j])[c / 2];
            wv = c % 2 ? E::hi(w2) : E::lo(w2);
        }
        if constexpr (u % 4 == 1) part[0] = fmaf(wv, wv, e % 16 ? part[0] : 0.f);
        if constexpr (u % 4 == 2) part[1] = fmaf(wv, v, e % 16 ? part[1] : 0.f);
        if constexpr (u % 4 == 3) part[2] = fmaf(v, v, e % 16 ? part[2] : 0.f);
        if constexpr (u % 64 == 63) {
#pragma unroll
            for (int k = 0; k < 3; ++k) sum[k][i] += part[k];
        }
    };
    auto read_w = [&](auto n_tag, uint32_t slot0, uint32_t slot1) {    // rows 16 (n / 4) .. of the wave, column block n % 4
        constexpr int n = decltype(n_tag)::value;
        w[n / 4][n % 4] = lds_read_b64<n / 4 % 2 * 2048>((n / 8 ? slot1 : slot0) + rwd[n % 4]);
    };
    auto w_landed = [](auto n_tag, uint64_t (&v)[4][4]) {   // all but the last N reads
        asm volatile("s_waitcnt lgkmcnt(%16)" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[0][3]), "+v"(v[1][0]), "+v"(v[1][1]),
                     "+v"(v[1][2]), "+v"(v[1][3]), "+v"(v[2][0]), "+v"(v[2][1]), "+v"(v[2][2]), "+v"(v[2][3]), "+v"(v[3][0]),
                     "+v"(v[3][1]), "+v"(v[3][2]), "+v"(v[3][3]) : "n"(decltype(n_tag)::value));
    };
    // Fragments of a half step (32 k) and of the next.  The products go column block by column block; once those of block j
    // of half step h are under way (behind the first of the next block), block j of half step h + 2 is read into its
    // registers.  So before the products of any block the last six reads (twelve instructions) are of later ones.
    bf16x8_t frag[2][4];
    auto read_frag = [&](auto h_tag, auto j_tag, uint32_t slot) {      // half H of a K step
        constexpr int H = decltype(h_tag)::value, j = decltype(j_tag)::value;
        frag[H][j] = lds_read_tr<H * 32 * BN * 2, 4 * BN * 2>(slot + rb[j]);
    };
    auto frag_landed = [](bf16x8_t& f) { asm volatile("s_waitcnt lgkmcnt(12)" : "+v"(f)); };
    int pos = 0;                                       // ring position of the K step under way
    auto behind = [&](int n) { const int q = pos + n; return q >= NS ? q - NS : q; };   // 0 <= n <= NS
    f32x4_t acc[4][4];
    auto keep = [&](int i, int j) {
        asm volatile("" : "+a"(acc[i][j]));
        old[i][j] = acc[i][j];
        asm volatile("" : "+v"(old[i][j]));
    };

    // column tile t; OLD: there is a tile before it, whose products are still in acc
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 3> I3;
    auto tile = [&](auto old_tag, int t) {
        constexpr bool OLD = decltype(old_tag)::value;
        uint32_t slot = 0;                             // of the next K step
        static_for<2 * S>([&](auto ht) {
            constexpr int h = decltype(ht)::value, s = h / 2, H = h % 2;
            const uint32_t w0 = (uint32_t)behind(NS - 2) * SLOT, w1 = (uint32_t)behind(NS - 1) * SLOT;   // W of the tile before
            if constexpr (OLD && h == 1) w_landed(std::integral_constant<int, 4>{}, w);
            static_for<16>([&](auto nt) {
                constexpr int n = decltype(nt)::value, i = n % 4, j = n / 4;
                if constexpr (i == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    frag_landed(frag[H][j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (H == 0 && n == 4) {
                    // The next K step (of the next tile: past the two slots of W) has landed, and everyone has read what is
                    // refilled up to the next such point.
                    constexpr int AHEAD = s == S - 1 ? 3 : 1;
                    wait_vmcnt<Refill<S, NS>::loads_before(h * 16 + n) - (s + AHEAD + 1) * LPS>();
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                    slot = (uint32_t)behind(AHEAD) * SLOT;
                }
                if constexpr (OLD && h == 0) keep(i, j);
                acc[i][j] = E::mfma16(frag[H][j], bf[h][i], h == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[i][j]);
                if constexpr (OLD && h == 0 && n < 8) {
                    read_w(std::integral_constant<int, 2 * n>{}, w0, w1);
                    read_w(std::integral_constant<int, 2 * n + 1>{}, w0, w1);
                }
                if constexpr (n == 0) read_frag(std::integral_constant<int, 1 - H>{}, I3{}, H == 0 ? (uint32_t)pos * SLOT : slot);
                else if constexpr (i == 0) read_frag(std::integral_constant<int, H>{}, std::integral_constant<int, j - 1>{}, slot);
                if constexpr (Refill<S, NS>::load_at(h * 16 + n) >= 0) {
                    constexpr int k = Refill<S, NS>::load_at(h * 16 + n), seq = k / LPS;
                    walk.template issue_one<seq, k % LPS>(t, smem + behind((seq - s) % NS) * SLOT);
                }
                if constexpr (OLD && h > 0) {
                    constexpr int N = (2 * S - 1) * 16, m = (h - 1) * 16 + n, u0 = m * 256 / N, u1 = (m + 1) * 256 / N;
                    static_for<u1 - u0>([&](auto ut) { sums(std::integral_constant<int, u0 + decltype(ut)::value>{}); });
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (H == 1) pos = behind(s == S - 1 ? 3 : 1);
        });
    };
    wait_vmcnt<(FIRST - 1) * LPS>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_frag(I0{}, I0{}, 0u); read_frag(I0{}, I1{}, 0u); read_frag(I0{}, I2{}, 0u); read_frag(I0{}, I3{}, 0u);
    read_frag(I1{}, I0{}, 0u); read_frag(I1{}, I1{}, 0u); read_frag(I1{}, I2{}, 0u);
    tile(std::integral_constant<bool, false>{}, walk.t_begin);
    for (int t = walk.t_begin + 1; t < walk.t_end; ++t) tile(std::integral_constant<bool, true>{}, t);
    // the last tile's sums (the fragments read past it keep their registers until they have landed)
    static_for<16>([&](auto nt) {
        constexpr int n = decltype(nt)::value;
        keep(n / 4, n % 4);
        read_w(nt, (uint32_t)behind(NS - 2) * SLOT, (uint32_t)behind(NS - 1) * SLOT);
    });
    w_landed(I0{}, w);
#pragma unroll
    for (int q = 0; q < 2; ++q) asm volatile("" : "+v"(frag[q][0]), "+v"(frag[q][1]), "+v"(frag[q][2]), "+v"(frag[q][3]));
    __builtin_amdgcn_sched_barrier(0);
    static_for<256>([&](auto ut) { sums(ut); });
    wait_vmcnt<0>();                                   // the loads past the end have written their zeros
    store_sums(p, reinterpret_cast<float*>(smem), sum, wave, lane, walk.slice, walk.m0, rows);
}

template <int DT>
hipError_t launch(const NormRowsArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.d_out + BM - 1) / BM * a.slices)), block(256);
    switch ((a.r + 63) / 64) {
        case 1: norm_rows_kernel<1, DT><<<grid, block, 0, st>>>(a); break;
        case 2: norm_rows_kernel<2, DT><<<grid, block, 0, st>>>(a); break;
        case 3: norm_rows_deep_kernel<3, DT><<<grid, block, 0, st>>>(a); break;
        case 4: norm_rows_deep_kernel<4, DT><<<grid, block, 0, st>>>(a); break;
        case 5: norm_rows_deep_kernel<5, DT><<<grid, block, 0, st>>>(a); break;
        case 6: norm_rows_deep_kernel<6, DT><<<grid, block, 0, st>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_norm_rows(const NormRowsArgs& a, int dt, hipStream_t st)
{
    TraceScope ts(DORA_K_NORM_CROSS, st);
    return dt == DT_F16 ? launch<DT_F16>(a, st) : launch<DT_BF16>(a, st);
}

}  // namespace dora
