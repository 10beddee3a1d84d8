// Forward of a few tokens (decode): every product streams its weight matrix once and multiplies it with a handful
// of token rows, so the launches are bound by reading W (2 d_out d_in bytes) and by their own latency, not by MFMAs.
//
//   few_tokens_kernel<..., FINAL = false>   h = x A^T, K cut over workgroups and waves, fp32 slices to scratch
//   few_tokens_kernel<..., FINAL = true>    y = g (.) (x W^T + s h B^T) (+ bias), g = m / max(c, eps) formed here, h summed
//                                           from its slices; optionally inner and the saved h
//
// The 128 x 128 tiles of the other products would give such a call d_out / 128 workgroups (32 for 256 CUs at
// d_out = 4096).  Here a workgroup owns 16, 32 or 64 weight rows and its four waves split K, each streaming its own
// share through a private LDS ring (buffer_load ... lds, 128-byte row segments, no barrier: only its own vmcnt), the
// token rows beside them in the same ring; the four partial tiles meet in LDS at the end.
#include "few_tokens_loads.hpp"
#include "lds_tile.hpp"

namespace dora {
namespace {

constexpr int WAVES = 4;
constexpr int STEP_K = FewTokensLoads<1, 1>::STEP_K;   // k per ring slot: row segments of one 128-byte line (256-byte ones measured the same)

// 16 bytes per lane from memory into 1 KB of LDS
__device__ __forceinline__ void load_1k(char* lds, __amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t soffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_ptr_t)lds, 16, off, soffset, 0, 0);
}

// TB: blocks of 16 tokens; MR: blocks of 16 weight rows; DEPTH: ring slots of a wave
template <int TB, int MR, int DEPTH, bool FINAL, int DT, bool LOW_RANK = false>
__global__ __launch_bounds__(64 * WAVES) void few_tokens_kernel(FewTokensArgs p)
{
    typedef Elem16<DT> E;
    typedef FewTokensLoads<TB, MR> L;
    constexpr int ROWS = L::ROWS, TOK = L::TOK;
    constexpr int SLOT_BYTES = (ROWS + TOK) * STEP_K * 2;
    constexpr int LPS = L::COUNT;                      // wave-wide loads per ring slot
    constexpr int LPB = 16 / L::LOAD_ROWS;             // of them per block of 16 rows
    constexpr int KSTEPS = STEP_K / 32;                // MFMA k-steps per ring slot
    constexpr int RED_LD = ROWS + 4;
    constexpr int RING_BYTES = WAVES * DEPTH * SLOT_BYTES, RED_BYTES = WAVES * TOK * RED_LD * 4;
    constexpr int LDS_BYTES = RING_BYTES > RED_BYTES ? RING_BYTES : RED_BYTES;
    // One block of tokens and of rows: h comes through LDS, H_RANKS of it at a time.  Up to one k-step of it to a wave (LOW_RANK) the
    // waves take their own as they are: six shapes of 512 x 512 to 8192 x 2048, forward of 1 to 16 tokens, r 8 1.07 times faster than
    // through LDS, r 64 1.05, r 128 1.00 to 1.04, r 256 1.05 to 1.10.  (512 x 512, r 8, 1 token 6.6 us through LDS, whose loads are
    // issued for all slices by every wave, 5.8 this way; 4096 x 4096, r 384 in LDS 14.1, from memory 20.3, weights from HBM.)
    constexpr bool STAGE_H = FINAL && TB == 1 && MR == 1 && !LOW_RANK, DIRECT_H = FINAL && LOW_RANK;
    static_assert(!LOW_RANK || (TB == 1 && MR == 1), "a wave's own k-step of one block");
    constexpr int H_RANKS = 512, H_BYTES = STAGE_H ? 16 * H_RANKS * 2 : 0;
    static_assert(LDS_BYTES + H_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
    static_assert((DEPTH - 1) * LPS <= 63, "vmcnt is a 6-bit counter");
    __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES + H_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int group = (int)blockIdx.x / p.ksplit, z = (int)blockIdx.x % p.ksplit;
    const int n0 = group * ROWS;
    const int T = p.T, N = p.N, K = p.K;

    // this wave's share of the K steps
    const int steps = (K + STEP_K - 1) / STEP_K;
    const int parts = p.ksplit * WAVES, part = z * WAVES + wave;
    const int s_begin = (int)((int64_t)steps * part / parts), s_end = (int)((int64_t)steps * (part + 1) / parts);

    // descriptors of the weight rows of this group and of the token rows
    const int w_rows = N - n0 < ROWS ? N - n0 : ROWS;
    __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.w + (int64_t)n0 * K), 0,
                                                                  (int)(uint32_t)((int64_t)w_rows * K * 2), 0x00020000);
    __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.x), 0, (int)(uint32_t)((int64_t)T * K * 2),
                                                                  0x00020000);
    // per-lane offsets of a slot's loads at k0 = 0; the swizzle, and with it k, repeats every 16 rows
    uint32_t vo[LPS];
    int kl[LPB];
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
        const int row = L::row(i, lane);
        const int k = ((lane % L::LANES_PER_ROW) ^ kc_swizzle<STEP_K>(row)) * 8;
        vo[i] = L::vector_offset(row, L::weights(i) ? w_rows : T, k, K);
        if (i < LPB) kl[i] = k;
    }
    char* const ring = smem + wave * (DEPTH * SLOT_BYTES);
    auto issue = [&](int s, int slot) {
        char* tile = ring + slot * SLOT_BYTES;
        const int k0 = s * STEP_K;
        const int k_end = s < s_end ? K : 0;           // a step past this wave's share brings zeros
        auto load_slot = [&](auto&& offset) {
            static_for<LPS>([&](auto it) {
                constexpr int i = decltype(it)::value;
                load_1k(tile + i * 1024, L::weights(i) ? rw : rx, offset(i), L::scalar_offset(k0));
            });
        };
        // whole steps take their offsets as they are (masked every time, 122 shapes take 0.6 % longer on average)
        if (k0 + STEP_K <= k_end) load_slot([&](int i) { return vo[i]; });
        else load_slot([&](int i) { return L::step_offset(vo[i], kl[i % LPB], k0, k_end); });
    };

    f32x4_t acc[MR][TB], accl[MR][TB];
#pragma unroll
    for (int i = 0; i < MR; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[i][j][e] = 0.f; accl[i][j][e] = 0.f; }

    typedef __attribute__((address_space(3))) const char* lds_cptr_t;
    constexpr int PAIRS = ROWS / 2;
    static_assert(64 * WAVES % PAIRS == 0, "a thread keeps its columns");
    const int c_own = (int)threadIdx.x % PAIRS * 2, n_own = n0 + c_own;     // the two columns this thread stores in the end
    float2 cj = make_float2(1.f, 1.f), mj = make_float2(0.f, 0.f);
    uint32_t bias = 0u;
    // Everything the low-rank part and the end need is asked for ahead of the first weight rows: loads complete in order, and
    // one latency covers them all.  (Each slice of h waited for the one before, k-step after k-step, behind the first weight
    // rows, and g's norm and magnitude for the end: forward of 4096 x 4096, r 384, weights from memory, 1 token 20.3 -> 14.1 us,
    // 16 tokens 23.2 -> 17.1, 64, whose h stays out of LDS, 34.3 -> 29.4; with W left in a cache by the call before, 1 token, this
    // launch alone 14.7 -> 9.0.)
    constexpr int SLICES = 8 / TB;                     // slices of h at most (few_tokens_h_slices)
    // all of NS slices are asked for (the last one again past the end: cheaper than a branch at each), summed in slice order and
    // rounded once to the storage type, as the saved tensor is
    typedef std::integral_constant<int, SLICES> All;
    typedef std::integral_constant<int, 1> One;
    float4 hs[SLICES][2];                              // of the k-step or item under way
    auto load_h = [&](auto ns, int t, int l, float4 (&v)[decltype(ns)::value][2]) {
#pragma unroll
        for (int z = 0; z < decltype(ns)::value; ++z) {
            if (DIRECT_H && z >= p.h_slices) continue;
            const int zz = z < p.h_slices ? z : p.h_slices - 1;
            const float4* hp = reinterpret_cast<const float4*>(p.h_part + ((int64_t)zz * T + t) * p.r + l);
            v[z][0] = hp[0]; v[z][1] = hp[1];
        }
    };
    auto sum_h = [&](auto ns, const float4 (&v)[decltype(ns)::value][2]) {
        float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int z = 0; z < decltype(ns)::value; ++z)
            if (z < p.h_slices) {
                a[0] += v[z][0].x; a[1] += v[z][0].y; a[2] += v[z][0].z; a[3] += v[z][0].w;
                a[4] += v[z][1].x; a[5] += v[z][1].y; a[6] += v[z][1].z; a[7] += v[z][1].w;
            }
        uint4 o;
        o.x = E::pack2(a[0], a[1]); o.y = E::pack2(a[2], a[3]); o.z = E::pack2(a[4], a[5]); o.w = E::pack2(a[6], a[7]);
        return o;
    };
    auto load_b = [&](int i, int l) {
        const int n = n0 + i * 16 + l16;
        uint4 b = make_uint4(0u, 0u, 0u, 0u);
        if (l < p.r && n < N) b = *reinterpret_cast<const uint4*>(p.b + (int64_t)n * p.r + l);
        return b;
    };
    constexpr int PRE = H_RANKS / 32 / WAVES;          // k-steps of a wave in H_RANKS
    uint4 bpre[STAGE_H ? PRE : 1];
    const bool own_step = wave * 32 < p.r;             // DIRECT_H: this wave's
    // item of h: eight ranks of one token; `per` of them to a token, ranks past r among them as far as a k-step reaches
    const int per0 = ((p.r < H_RANKS ? p.r : H_RANKS) + 31) / 32 * 4;
    if constexpr (FINAL) {
        if (n_own < N) {
            cj = *reinterpret_cast<const float2*>(p.c + n_own);
            mj = *reinterpret_cast<const float2*>(p.m + n_own);
            if (p.bias) bias = *reinterpret_cast<const uint32_t*>(p.bias + n_own);
        }
        if constexpr (STAGE_H) {
            const int t = (int)threadIdx.x / per0, l = (int)threadIdx.x % per0 * 8;
            load_h(All{}, t < T ? t : T - 1, l < p.r ? l : 0, hs);
#pragma unroll
            for (int q = 0; q < PRE; ++q) bpre[q] = load_b(0, (wave + q * WAVES) * 32 + lq * 8);
        }
        if constexpr (DIRECT_H) {
            const int l = wave * 32 + lq * 8;
            if (own_step && l16 < T) load_h(All{}, l16, l < p.r ? l : 0, hs);
            if (own_step) bpre[0] = load_b(0, l);
        }
        __builtin_amdgcn_sched_barrier(0);
    }

#pragma unroll
    for (int d = 0; d < DEPTH; ++d) issue(s_begin + d, d);
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (STAGE_H) {
        const uint32_t hbuf = (uint32_t)(uintptr_t)(lds_cptr_t)(smem + LDS_BYTES);
        for (int c0 = 0; c0 < p.r; c0 += H_RANKS) {
            const int left = p.r - c0, per = ((left < H_RANKS ? left : H_RANKS) + 31) / 32 * 4;
            if (c0 > 0) {
#pragma unroll
                for (int q = 0; q < PRE; ++q) bpre[q] = load_b(0, c0 + (wave + q * WAVES) * 32 + lq * 8);
            }
            for (int i = threadIdx.x; i < T * per; i += 64 * WAVES) {
                const int t = i / per, k = i % per * 8, l = c0 + k;
                if (c0 > 0 || i >= 64 * WAVES) load_h(All{}, t, l < p.r ? l : 0, hs);
                uint4 o = sum_h(All{}, hs);
                if (l >= p.r) o = make_uint4(0u, 0u, 0u, 0u);
                if (p.h_out && blockIdx.x == 0 && l < p.r) *reinterpret_cast<uint4*>(p.h_out + (int64_t)t * p.r + l) = o;
                const uint32_t at = hbuf + (uint32_t)(t * (H_RANKS * 2) + (((k >> 3) ^ t) << 4));
                asm volatile("ds_write_b128 %0, %1" ::"v"(at), "v"(__builtin_bit_cast(bf16x8_t, o)) : "memory");
            }
            wait_lgkmcnt<0>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < PRE; ++q) {
                const int st = wave + q * WAVES;
                if (st * 32 >= left) continue;
                // (tokens past T: whatever is there reaches only columns that are not stored)
                bf16x8_t hf = lds_read_b128<0>(hbuf + (uint32_t)(l16 * (H_RANKS * 2) + (((st * 4 + lq) ^ l16) << 4)));
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(hf));
                accl[0][0] = E::mfma16(__builtin_bit_cast(bf16x8_t, bpre[q]), hf, accl[0][0]);
            }
            __builtin_amdgcn_s_barrier();              // read by all: the next ranks, or the ring, may follow
            __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (DIRECT_H) {
        const int l = wave * 32 + lq * 8;
        if (own_step) {
            uint4 o = sum_h(All{}, hs);                    // (tokens past T: whatever is there reaches only columns that are not stored)
            if (l >= p.r) o = make_uint4(0u, 0u, 0u, 0u);
            if (p.h_out && blockIdx.x == 0 && l < p.r && l16 < T) *reinterpret_cast<uint4*>(p.h_out + (int64_t)l16 * p.r + l) = o;
            accl[0][0] = E::mfma16(__builtin_bit_cast(bf16x8_t, bpre[0]), __builtin_bit_cast(bf16x8_t, o), accl[0][0]);
        }
    } else if constexpr (FINAL) {
        // low-rank part while the first weight rows are on their way: h and B straight from memory, the waves share the
        // k-steps of 32.  One slice of h, of a short d_in, is not asked for SLICES times (weights from memory: 7760 x 200, r 464,
        // 32 tokens 16.6 us, 11.0 this way; 4096 x 512, r 512 15.3, 10.1)
        auto low_rank = [&](auto ns) {
            for (int st = wave; st * 32 < p.r; st += WAVES) {
                const int l = st * 32 + lq * 8;
                const bool ok = l < p.r;
                bf16x8_t hf[TB], bfr[MR];
                float4 v[TB][decltype(ns)::value][2];
#pragma unroll
                for (int j = 0; j < TB; ++j) {
                    const int t = j * 16 + l16;
                    load_h(ns, t < T ? t : T - 1, ok ? l : 0, v[j]);
                }
#pragma unroll
                for (int i = 0; i < MR; ++i) bfr[i] = __builtin_bit_cast(bf16x8_t, load_b(i, l));
#pragma unroll
                for (int j = 0; j < TB; ++j) {
                    const int t = j * 16 + l16;
                    uint4 o = sum_h(ns, v[j]);
                    if (!ok) o = make_uint4(0u, 0u, 0u, 0u);
                    hf[j] = __builtin_bit_cast(bf16x8_t, o);
                    if (p.h_out && blockIdx.x == 0 && ok && t < T) *reinterpret_cast<uint4*>(p.h_out + (int64_t)t * p.r + l) = o;
                }
#pragma unroll
                for (int i = 0; i < MR; ++i)
#pragma unroll
                    for (int j = 0; j < TB; ++j) accl[i][j] = E::mfma16(bfr[i], hf[j], accl[i][j]);
            }
        };
        if (__builtin_expect(p.h_slices > 1, 1)) low_rank(All{});
        else low_rank(One{});
    }

    const uint32_t ring_lds = (uint32_t)(uintptr_t)(lds_cptr_t)ring;
    uint32_t rd[KSTEPS];
#pragma unroll
    for (int q = 0; q < KSTEPS; ++q)
        rd[q] = ring_lds + (uint32_t)lds_off<STEP_K>(l16, q * 32 + lq * 8);
    int slot = 0;
    for (int s = s_begin; s < s_end; ++s) {
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt<(DEPTH - 1) * LPS>();               // the oldest slot has landed
        __builtin_amdgcn_sched_barrier(0);
        bf16x8_t f[KSTEPS][MR + TB];
        static_for<KSTEPS * (MR + TB)>([&](auto it) {
            constexpr int q = decltype(it)::value / (MR + TB), b = decltype(it)::value % (MR + TB);
            f[q][b] = lds_read_b128<b * 16 * STEP_K * 2>(rd[q] + slot * SLOT_BYTES);
        });
        wait_lgkmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        issue(s + DEPTH, slot);                        // its reads are done: refill it
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < KSTEPS; ++q)
#pragma unroll
            for (int i = 0; i < MR; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j) acc[i][j] = E::mfma16(f[q][i], f[q][MR + j], acc[i][j]);
        slot = slot + 1 == DEPTH ? 0 : slot + 1;
    }
    wait_vmcnt<0>();                                   // the loads past the end have written their zeros
    __syncthreads();

    // lane: weight rows 4 lq .. +3 of block i, token l16 of block j.  The four waves' tiles meet in LDS.
    float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < MR; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            float4 v = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            if constexpr (FINAL) {
                v.x = fmaf(p.s, accl[i][j][0], v.x); v.y = fmaf(p.s, accl[i][j][1], v.y);
                v.z = fmaf(p.s, accl[i][j][2], v.z); v.w = fmaf(p.s, accl[i][j][3], v.w);
            }
            *reinterpret_cast<float4*>(red + (wave * TOK + j * 16 + l16) * RED_LD + i * 16 + lq * 4) = v;
        }
    __syncthreads();
    for (int e = threadIdx.x; e < TOK * PAIRS; e += 64 * WAVES) {
        const int t = e / PAIRS;
        if (t >= T || n_own >= N) continue;            // N is a multiple of 8
        float v0 = 0.f, v1 = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float2 u = *reinterpret_cast<const float2*>(red + (w * TOK + t) * RED_LD + c_own);
            v0 += u.x; v1 += u.y;
        }
        if constexpr (FINAL) {
            const float g0 = mj.x / ((cj.x < p.eps) ? p.eps : cj.x), g1 = mj.y / ((cj.y < p.eps) ? p.eps : cj.y);
            const int64_t at = (int64_t)t * N + n_own;
            *reinterpret_cast<uint32_t*>(p.y + at) = E::pack2(fmaf(g0, v0, E::lo(bias)), fmaf(g1, v1, E::hi(bias)));
            if (p.inner) *reinterpret_cast<uint32_t*>(p.inner + at) = E::pack2(v0, v1);
        } else {
            *reinterpret_cast<float2*>(p.part + ((int64_t)z * T + t) * N + n_own) = make_float2(v0, v1);
        }
    }
}

// Ring depth and rows per workgroup: us of a forward in bf16, one after the other over as many sets of weights and inputs as
// make 600 MB, so that no set is left in a cache from its last turn.
//  - Up to 8192 weight rows 16 of them make at most 512 workgroups, two per CU in one go, and a shallow ring that lets two
//    share a CU beats a deep one (1 token at 8192 x 8192, r 768 47.7 against 59.9 for eight slots, at 4104 x 4096, r 64
//    15.4 / 20.5) and workgroups of 64 rows (8192 x 4096, r 64, 1 and 32 tokens 20.0 and 27.7 / 23.8 and 29.4).
//  - Beyond, 16 rows would need a second round, and 64 rows win from the first row on (8200 x 4096, r 64 24.0 and 29.1 / 25.5
//    and 32.4, 10240 24.8 and 31.1 / 29.7 and 36.9, 14336 28.7 and 32.7 / 32.5 and 44.9); the token rows are then re-read for
//    a quarter as many workgroups.
//  - With four token blocks that re-reading asks for 32 rows above 4096 of them (64 tokens at 4104 x 4096, r 64 27.9 / 32.8
//    for 16 rows, 8192 x 4096 32.3 / 37.2), not at 4096 (r 384 34.4 / 37.1 the other way round).
template <int DT>
hipError_t launch_y(const FewTokensArgs& a, hipStream_t st)
{
    const bool narrow = a.N <= 4096, wide = a.N > 8192;
#define DORA_FEW(TB, MR, DEPTH) \
    few_tokens_kernel<TB, MR, DEPTH, true, DT><<<dim3((unsigned)((a.N + MR * 16 - 1) / (MR * 16))), dim3(64 * WAVES), 0, st>>>(a)
    if (a.T <= 16 && !wide && a.r <= 32 * WAVES)
        few_tokens_kernel<1, 1, 4, true, DT, true><<<dim3((unsigned)((a.N + 15) / 16)), dim3(64 * WAVES), 0, st>>>(a);
    else if (a.T <= 16) { if (wide) DORA_FEW(1, 4, 2); else DORA_FEW(1, 1, 4); }
    else if (a.T <= 32) { if (wide) DORA_FEW(2, 4, 2); else DORA_FEW(2, 1, 3); }
    else if (wide) DORA_FEW(4, 4, 2);
    else if (narrow) DORA_FEW(4, 1, 2);
    else DORA_FEW(4, 2, 2);
#undef DORA_FEW
    return hipGetLastError();
}

template <int DT>
hipError_t launch_h(const FewTokensArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.N + 15) / 16 * a.ksplit)), block(64 * WAVES);
    if (a.T <= 16) few_tokens_kernel<1, 1, 4, false, DT><<<grid, block, 0, st>>>(a);
    else if (a.T <= 32) few_tokens_kernel<2, 1, 3, false, DT><<<grid, block, 0, st>>>(a);
    else few_tokens_kernel<4, 1, 2, false, DT><<<grid, block, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace

// Slices of d_in for h = x A^T: r / 16 workgroups leave most of the chip idle, but every workgroup of the y launch sums
// all slices of all tokens again, so few of them where there are many tokens, and two ring slots per wave at least.
int few_tokens_h_slices(int64_t tokens, int64_t r, int64_t d_in)
{
    const int64_t groups = (r + 15) / 16;
    const int64_t tb = (tokens + 15) / 16, steps = (d_in + STEP_K - 1) / STEP_K;
    int64_t ks = 256 / groups;
    if (ks > 8 / tb) ks = 8 / tb;
    if (ks > steps / (2 * WAVES)) ks = steps / (2 * WAVES);
    return ks < 1 ? 1 : (int)ks;
}

hipError_t launch_few_tokens_h(const FewTokensArgs& a, int dt, hipStream_t st)
{
    TraceScope ts(DORA_K_GEMM_H, st);
    return dt == DT_F16 ? launch_h<DT_F16>(a, st) : launch_h<DT_BF16>(a, st);
}

hipError_t launch_few_tokens_y(const FewTokensArgs& a, int dt, hipStream_t st)
{
    TraceScope ts(DORA_K_GEMM_FUSED_FWD, st);
    return dt == DT_F16 ? launch_y<DT_F16>(a, st) : launch_y<DT_BF16>(a, st);
}

}  // namespace dora
