// Chunk attention for steps of many query rows (gfx950, bf16 caches): prompts,
// prefixes and catch-up chunks, whose G * n_q query rows of a KV head fill more
// than one 128-row workgroup.
//
//   attn_block  one workgroup = (block of 128 query rows, key split, KV head,
//               stream), 8 waves: wave w takes the 32 rows w % 4 and every second
//               64-key tile (w / 4); the two key halves' states are combined in
//               LDS at the end.  The step's rows are already in the cache
//               (append_kernel runs first), so every key tile is read the same way.
//
// Bound: matrix and vector ALU together, and the tiles' way from L2 into LDS.  A
// wave's tile is 32 v_mfma_f32_32x32x16_bf16 at head dim 128 (1024 cycles) and 32
// elements of softmax per lane (~900 cycles); the two waves of a SIMD overlap one's
// products with the other's softmax.  32-row waves read each K and V operand from
// LDS once for 32 query rows; the key halves give a SIMD its second wave where the
// query blocks alone are one workgroup per CU (1,024 rows x 4 heads x 8 KV heads).
// Measured there (head dim 128, 5,120 keys, 77 GFLOP a layer): 86 us, 0.90 PFLOP/s, the
// matrix units busy 36 % of it (attn_tile with 27 key splits and their merge: 482 us).  Of
// variants timed when it took 82 us: with no tile DMA after the first step 69 us; one wave
// of 64 rows per SIMD 123, one of 32 rows x 64 keys 125, the halves held in opposite
// phases by barriers 83 (and 18 instead of 15.5 us on a 777-row prompt at head dim 64).
#include "a2t_internal.h"
#include "device_common.h"

#include <hip/hip_ext.h>

#include <type_traits>

namespace a2t {
namespace {

constexpr int kBlockThreads = 512;
constexpr int kWaveRows = 32;
static_assert(kWaveRows * 4 == kBlockRows && kBlockThreads == 512, "four row groups x two key halves");

typedef float f32x16 __attribute__((ext_vector_type(16)));

// s_waitcnt lgkmcnt(N) that the listed LDS reads depend on (LDS reads complete
// in order: with N reads issued after them these are complete)
template <int N>
__device__ __forceinline__ void lds_wait(u32x4 (&a)[8]) {
    asm volatile("s_waitcnt lgkmcnt(%8)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
                 : "i"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x4 (&a)[4]) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "i"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait(uint2 (&a)[8]) {
    asm volatile("s_waitcnt lgkmcnt(%8)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
                 : "i"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait(uint2 (&a)[4]) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "i"(N));
}

// max / sum over the two lanes l, l ^ 32 that hold one query column
__device__ __forceinline__ float pair_max(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// S^T = K.Q^T: A = K rows (32 keys x 16 dims), B = Q^T (16 dims x 32 queries);
// lane l (h = l / 32) gets, for query l % 32, keys 8 (r / 4) + 4 h + r % 4 of the
// 32-key block in accumulator register r.  Eight consecutive registers are then
// the B operand of O^T = V^T.P^T for 16 keys, with k-slot 8 h + j holding key
// 8 (j / 4) + 4 h + j % 4; the A operand reads the same keys of V with two
// transposed LDS reads.
//
// The 16-byte chunks of a tile row are stored swizzled so that neither read has a
// bank conflict: the 16 rows that a quarter of a K read touches lie in 16 different
// chunk places of 256 bytes, and so do the four rows x 64 bytes that half of a
// transposed V read touches.
template <int D>
__device__ __forceinline__ int k_swizzle(int row) {
    return D == 128 ? row & 15 : (row >> 1) & 7;
}
template <int D>
__device__ __forceinline__ int v_swizzle(int row) {
    return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1);
}

template <int D, int N>
__global__ __launch_bounds__(kBlockThreads) void attn_block_kernel(DevState st, AttnBatchT<N> b, WgStart<N> start,
                                                                   const uint16_t* q, uint16_t* o) {
    constexpr int KS = D / 16;                 // k-steps of Q.K^T
    constexpr int DB = D / 32;                 // 32-dim blocks of O
    constexpr int CPR = D / 8;                 // 16-byte chunks per row
    constexpr int RPB = 512 / D;               // rows per 1 KiB DMA block
    constexpr int OPS = kTileKeys / RPB / 4;   // K (and V) DMA blocks per wave and tile
    constexpr int TILE = kTileKeys * D;
    __shared__ __align__(1024) uint16_t ring[8 * TILE];   // per key half two K and two V stages
    __shared__ float2 s_ml[4][64];
    static_assert(8 * TILE * 2 >= 4 * DB * 16 * 256, "the second key half's sums fit the ring");

    int wg;
    const AttnDesc d = b.d[stream_of(start, b.count, &wg)];
    const int G = st.G, nq = d.n_q, M = G * nq, R = d.R;
    const int nqb = (M + kBlockRows - 1) / kBlockRows;
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };   // divisions run on the vector ALU
    // linear block (split, query block, KV head), heads fastest: the workgroups of
    // a head share an XCD's L2 when the head count divides the 8 XCDs, and the
    // later query blocks, which see the most keys, are dispatched first
    const int y = uniform(wg / st.Hkv), g = wg - y * st.Hkv;
    const int sp = uniform(y / nqb), qb = nqb - 1 - (y - sp * nqb);
    if (sp >= d.splits) return;
    const int w = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
    const int l16 = lane & 15, lg = lane >> 4;
    const int rg = w & 3, kh = w >> 2;   // row group, key half
    const int mw = qb * kBlockRows + kWaveRows * rg;
    const int mq = mw + l32;             // this lane's query row
    const int vis0 = R - nq;
    // keys past the block's last row are masked for all its rows: their tiles are left out
    const int last_i = uniform((min(M, (qb + 1) * kBlockRows) - 1) / G);
    const int t_end = (vis0 + last_i) / kTileKeys + 1;
    const int t0 = sp * d.tile_q + min(sp, d.tile_r);
    const int t1 = min(t0 + d.tile_q + (sp < d.tile_r ? 1 : 0), t_end);
    const int kept = d.kept, head = d.head, ring_rows = st.unit_rows;

    const uint16_t* ku = reinterpret_cast<const uint16_t*>(st.k_unit) + pool_index(st, b.layer, d.s, g, ring_rows, 0);
    const uint16_t* vu = reinterpret_cast<const uint16_t*>(st.v_unit) + pool_index(st, b.layer, d.s, g, ring_rows, 0);
    // elements from a head's ring to its kept region, the same in both pools
    const int64_t to_kept = (reinterpret_cast<const uint16_t*>(st.k_kept) - reinterpret_cast<const uint16_t*>(st.k_unit)) +
                            pool_index(st, b.layer, d.s, g, st.kept_rows, 0) - pool_index(st, b.layer, d.s, g, ring_rows, 0);

    // A wave fills the 1 KiB blocks rg * OPS + i of a tile, rows (rg * OPS + i) * RPB ..;
    // lane j fills physical chunk j % CPR of row j / CPR of each.  Block i's byte
    // offset is 1 KiB further and, for K, its chunk's bit 2 flips with i.
    const int row0 = rg * OPS * RPB + lane / CPR;
    const uint32_t lane_k = (uint32_t)(row0 * D + ((lane % CPR) ^ k_swizzle<D>(row0)) * 8) * 2u;
    const uint32_t lane_v = (uint32_t)(row0 * D + ((lane % CPR) ^ v_swizzle<D>(row0)) * 8) * 2u;
    const int64_t to_v = vu - ku;   // elements (a pointer picked by the flag would live in scratch)
    const uint32_t lane_d = lane_v - lane_k;
    auto issue = [&](int t, int is_v, uint16_t* buf) {
        const int kb = t * kTileKeys;
        const uint16_t* rows = ku + is_v * to_v;
        const uint32_t lane_off = lane_k + is_v * lane_d, flip = 64 - 64 * is_v;
        buf += rg * OPS * 512;
        // where the tile's row 0 is when the whole tile is one run of resident rows
        bool run = false;
        int64_t off = 0;
        if (kb + kTileKeys <= R) {
            if (kb + kTileKeys <= kept) {
                off = to_kept + (int64_t)kb * D;
                run = true;
            } else if (kb >= kept) {
                int slot = head + (kb - kept);
                if (slot >= ring_rows) slot -= ring_rows;
                off = (int64_t)slot * D;
                run = slot + kTileKeys <= ring_rows;
            }
        }
        if (run) {
            const char* base = reinterpret_cast<const char*>(rows + off);
#pragma unroll
            for (int i = 0; i < OPS; ++i) dma16(base + ((lane_off ^ (flip * i)) + 1024u * i), buf + i * 512);
        } else {
#pragma unroll 1
            for (int i = 0; i < OPS; ++i) {
                const int j = min(kb + row0 + i * RPB, R - 1);   // rows past R read row R-1: masked keys
                int slot = head + (j - kept);
                if (slot >= ring_rows) slot -= ring_rows;
                const int64_t src = j < kept ? to_kept + (int64_t)j * D : (int64_t)slot * D;
                dma16(rows + src + ((lane_off ^ (flip * i)) & (2 * D - 1)) / 2, buf + i * 512);
            }
            asm volatile("" ::: "memory");   // keeps the two paths' DMAs apart
        }
    };
    static_assert((RPB == 4 && OPS == 4) || (RPB == 8 && OPS == 2), "the offsets of a wave's DMA blocks");
    // a key half's waves load and read their own tiles only: tile i of half kh is
    // t0 + 2 i + kh (the second half of an odd count has one less)
    const int n = (t1 - t0 + 1) / 2;
    uint16_t* const ring_k = ring + kh * 4 * TILE;   // two K stages, two V stages
    uint16_t* const ring_v = ring_k + 2 * TILE;
    // K and V of tile i, if it is in the range
    auto issue_kv = [&](int i) {
        const int t = t0 + 2 * i + kh;
        if (t < t1) {
#pragma unroll 1
            for (int x = 0; x < 2; ++x) issue(t, x, ring_k + (2 * x + (i & 1)) * TILE);
        }
    };
    issue_kv(0);

    // Q^T operand of the lane's row: rotated, scaled by scale * log2(e), bf16.  Rows
    // past M read row M - 1 and are zeroed.
    bf16x8 qop[KS];
    {
        const int mqc = min(mq, M - 1);
        const int i = mqc / G, hh = mqc - i * G;
        const uint16_t* qp = q + ((int64_t)(d.q_row0 + i) * st.Hq + g * G + hh) * D + 8 * h;
        const float2* cp = st.rope + ((int64_t)d.s * st.max_step_rows + d.rope_row0 + i) * (D / 2) + 8 * h;
        const float qs = mq < M ? st.scale_log2e : 0.f;
        uint4 raw[KS];
        float4 cs[KS / 2][4];
#pragma unroll
        for (int s = 0; s < KS; ++s) raw[s] = *reinterpret_cast<const uint4*>(qp + 16 * s);
#pragma unroll
        for (int s = 0; s < KS / 2; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) cs[s][e] = *reinterpret_cast<const float4*>(cp + 16 * s + 2 * e);
#pragma unroll
        for (int s = 0; s < KS / 2; ++s) {
            const uint32_t lw[4] = {raw[s].x, raw[s].y, raw[s].z, raw[s].w};
            const uint32_t hw[4] = {raw[s + KS / 2].x, raw[s + KS / 2].y, raw[s + KS / 2].z, raw[s + KS / 2].w};
            uint32_t ol[4], oh[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float4 c4 = cs[s][e];
                const float a0 = __uint_as_float(lw[e] << 16), a1 = __uint_as_float(lw[e] & 0xffff0000u);
                const float b0 = __uint_as_float(hw[e] << 16), b1 = __uint_as_float(hw[e] & 0xffff0000u);
                ol[e] = pack_bf16x2((a0 * c4.x - b0 * c4.y) * qs, (a1 * c4.z - b1 * c4.w) * qs);
                oh[e] = pack_bf16x2((b0 * c4.x + a0 * c4.y) * qs, (b1 * c4.z + a1 * c4.w) * qs);
            }
            qop[s] = __builtin_bit_cast(bf16x8, make_uint4(ol[0], ol[1], ol[2], ol[3]));
            qop[s + KS / 2] = __builtin_bit_cast(bf16x8, make_uint4(oh[0], oh[1], oh[2], oh[3]));
        }
    }

    // byte offsets of this lane's K operand of k-step 0 and of its transposed V reads of
    // dim block 0; k-step s and dim block db differ by an exclusive or
    const uint32_t koff = (uint32_t)(l32 * D + (h ^ k_swizzle<D>(l32)) * 8) * 2u;
    const int vr0 = 4 * (lg >> 1) + (l16 >> 2);   // rows 8 apart share vr0's swizzle
    const uint32_t voff = (uint32_t)(vr0 * D + ((2 * (lg & 1) + ((l16 & 3) >> 1)) ^ v_swizzle<D>(vr0)) * 8 + 4 * (l16 & 1)) * 2u;

    // mrun: the softmax reference of the lane's row (-inf: no visible key yet); the
    // products' accumulators start from -mu, so that scores come out relative to it
    float mrun = -INFINITY, mu = 0.f, lrun = 0.f, lrun1 = 0.f;
    f32x16 neg_mu;
#pragma unroll
    for (int r = 0; r < 16; ++r) neg_mu[r] = 0.f;
    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
    const int lim = vis0 + min(mq, M - 1) / G;              // last visible key of this lane's row
    const int lim_w = vis0 + uniform(min(mw, M - 1) / G);   // ... of the wave's first row

    // half of a tile's K operands: k-steps H * KS / 2 .., key blocks 0 and 1 in turn
    u32x4 ka[KS], kc[KS];
    auto k_issue = [&](const uint16_t* buf, auto half, u32x4 (&kop)[KS]) {
        constexpr int S0 = decltype(half)::value * (KS / 2);
        const uint32_t kb = lds_addr(buf) + koff;
#pragma unroll
        for (int e = 0; e < KS / 2; ++e) {
            kop[2 * e] = lds_b128_issue<0>(kb ^ (32 * (S0 + e)));
            kop[2 * e + 1] = lds_b128_issue<32 * D * 2>(kb ^ (32 * (S0 + e)));
        }
    };
    // the 16-key chunk C of V, rows 16 C + 0..7 and + 8..15 of each dim block
    auto v_issue = [&](const uint16_t* buf, auto chunk, uint2 (&vop)[2 * DB]) {
        constexpr int C = decltype(chunk)::value;
        const uint32_t vb = lds_addr(buf) + voff;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            vop[2 * db] = lds_tr16_issue<16 * C * D * 2>(vb ^ (64 * db));
            vop[2 * db + 1] = lds_tr16_issue<(16 * C + 8) * D * 2>(vb ^ (64 * db));
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    f32x16 sc[2];        // scores of the tile whose softmax comes next
    uint32_t pk[16];     // probabilities of the tile whose P.V comes next
    uint2 v0[2 * DB];    // its first chunk's V operands
    auto qk_half = [&](const u32x4 (&kop)[KS], int s0) {
#pragma unroll
        for (int e = 0; e < KS; ++e) {
            const f32x16 c = s0 + e / 2 == 0 ? neg_mu : sc[e & 1];
            sc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[e]), qop[s0 + e / 2], c, 0, 0, 0);
        }
    };
    auto pv = [&](const uint2 (&vop)[2 * DB], int c) {
        const bf16x8 p = __builtin_bit_cast(bf16x8, make_uint4(pk[4 * c], pk[4 * c + 1], pk[4 * c + 2], pk[4 * c + 3]));
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(vop[2 * db].x, vop[2 * db].y, vop[2 * db + 1].x, vop[2 * db + 1].y));
            acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p, acc[db], 0, 0, 0);
        }
    };
    auto softmax = [&](int t) {
        if (t * kTileKeys + kTileKeys - 1 > lim_w) {
            const int k0 = t * kTileKeys + 4 * h;
#pragma unroll
            for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (k0 + 32 * blk + 8 * (r >> 2) + (r & 3) > lim) sc[blk][r] = -INFINITY;
        }
        float m4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) m4[r] = fmaxf(sc[0][r], sc[1][r]);
#pragma unroll
        for (int r = 4; r < 16; ++r) m4[r & 3] = fmaxf(fmaxf(m4[r & 3], sc[0][r]), sc[1][r]);
        const float tmax = pair_max(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
        // the reference follows the row maximum lazily: raised (and the running sums
        // rescaled) only when a tile exceeds it by more than 2^8
        if (__any(tmax + mu > mrun + 8.f)) {
            const float mn = fmaxf(mrun, tmax + mu), ref = (mn == -INFINITY) ? 0.f : mn;
            const float corr = __builtin_amdgcn_exp2f(mrun - ref), shift = mu - ref;
            lrun *= corr;
            lrun1 *= corr;
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] *= corr;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sc[0][r] += shift;
                sc[1][r] += shift;
                neg_mu[r] = -ref;
            }
            mrun = mn;
            mu = ref;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float p0 = __builtin_amdgcn_exp2f(sc[i >> 3][(2 * i) & 15]);
            const float p1 = __builtin_amdgcn_exp2f(sc[i >> 3][(2 * i + 1) & 15]);
            lrun += p0;
            lrun1 += p1;
            pk[i] = pack_bf16x2(p0, p1);
        }
    };
    int stage = 0;
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        wait_vmem<0>();
        barrier_only();
        if (t0 + 2 * i + kh >= t1) break;   // the last round of an odd count
        k_issue(ring_k + stage * TILE, I0{}, ka);
        k_issue(ring_k + stage * TILE, I1{}, kc);
        issue_kv(i + 1);
        lds_wait<KS>(ka);
        qk_half(ka, 0);
        lds_wait<0>(kc);
        qk_half(kc, KS / 2);
        const uint16_t* vbuf = ring_v + stage * TILE;
        uint2 v1[2 * DB], v2[2 * DB], v3[2 * DB];
        // the first chunks' V operands are requested before the softmax
        v_issue(vbuf, I0{}, v0);
        v_issue(vbuf, I1{}, v1);
        asm volatile("" : "+v"(sc[0]), "+v"(sc[1]));
        softmax(t0 + 2 * i + kh);
        lds_wait<2 * DB>(v0);
        v_issue(vbuf, I2{}, v2);
        pv(v0, 0);
        lds_wait<2 * DB>(v1);
        v_issue(vbuf, I3{}, v3);
        pv(v1, 1);
        lds_wait<2 * DB>(v2);
        pv(v2, 2);
        lds_wait<0>(v3);
        pv(v3, 3);
        stage ^= 1;
    }
    __syncthreads();

    lrun += lrun1;
    // the second key half's sums through LDS (a lane of both halves holds the same
    // row and dims), combined and stored by the first half's waves
    float* part = reinterpret_cast<float*>(ring) + rg * (DB * 16 * 64) + lane;
    if (kh == 1) {
        s_ml[rg][lane] = make_float2(mrun, lrun);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) part[(db * 16 + r) * 64] = acc[db][r];
    }
    __syncthreads();
    if (kh == 1 || mw >= M) return;
    const float2 ml = s_ml[rg][lane];
    const float mn = fmaxf(mrun, ml.x), ref = (mn == -INFINITY) ? 0.f : mn;
    const float c0 = __builtin_amdgcn_exp2f(mrun - ref), c1 = __builtin_amdgcn_exp2f(ml.x - ref);
    const float ltot = pair_sum(lrun * c0 + ml.y * c1);
    // a row with no visible key in this split stores zeros with zero weight
    const float inv = (ltot == 0.f && d.splits > 1) ? 0.f : 1.f / ltot;
    const int i = mq / G, hh = mq - i * G;
    uint16_t* orow;
    if (d.splits > 1) {
        float* po = st.ws + d.ws_off;
        const int64_t at = ((int64_t)sp * st.Hkv + g) * M + mq;
        orow = reinterpret_cast<uint16_t*>(po) + at * D;
        if (h == 0 && mq < M)
            *reinterpret_cast<float2*>(po + (int64_t)d.splits * st.Hkv * M * (D / 2) + at * 2) = make_float2(mn, ltot);
    } else {
        orow = o + ((int64_t)(d.q_row0 + i) * st.Hq + g * G + hh) * D;
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[db][r] = (acc[db][r] * c0 + part[(db * 16 + r) * 64] * c1) * inv;
    // lanes l and l ^ 32 trade halves so that each lane stores 8 consecutive dims:
    // accumulator rows 8a + 4h .. + 3 of a pair of 8-dim groups (2a, 2a + 1) become
    // group 2a + h whole
    auto store = [&](auto pack) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                u32x4 out;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t u = pack(acc[db][8 * a + 2 * e], acc[db][8 * a + 2 * e + 1]);
                    const uint32_t v = pack(acc[db][8 * a + 4 + 2 * e], acc[db][8 * a + 4 + 2 * e + 1]);
                    const auto sw = __builtin_amdgcn_permlane32_swap(u, v, false, false);
                    out[e] = sw[0];
                    out[2 + e] = sw[1];
                }
                if (mq < M) *reinterpret_cast<u32x4*>(orow + 32 * db + 16 * a + 8 * h) = out;
            }
        }
    };
    // split partials: O / sum in fp16 (attn_merge_kernel), else the bf16 output
    if (d.splits > 1)
        store([](float x, float y) { return pack_f16x2(x, y); });
    else
        store([](float x, float y) { return pack_bf16x2(x, y); });
}

}  // namespace

hipError_t launch_attn_block(const DevState& st, const AttnBatch& b, const void* q, void* o, hipStream_t stream,
                             const KTimer& kt) {
    const uint16_t* qq = static_cast<const uint16_t*>(q);
    uint16_t* oo = static_cast<uint16_t*>(o);
    return by_size<AttnBatchT>(b, [&](const auto& bb) {
        constexpr int N = sizeof(bb.d) / sizeof(bb.d[0]);
        WgStart<N> start{};
        const dim3 grid = place_workgroups(b.count, &start, [&](int i) {
            return (st.G * b.d[i].n_q + kBlockRows - 1) / kBlockRows * b.d[i].splits * st.Hkv;
        });
        auto go = [&](auto kernel) {
            if (kt.start)
                hipExtLaunchKernelGGL(kernel, grid, dim3(kBlockThreads), 0, stream, kt.start, kt.stop, 0, st, bb, start, qq, oo);
            else
                hipLaunchKernelGGL(kernel, grid, dim3(kBlockThreads), 0, stream, st, bb, start, qq, oo);
            return hipGetLastError();
        };
        if (st.D == 128) return go(attn_block_kernel<128, N>);
        if (st.D == 64) return go(attn_block_kernel<64, N>);
        return hipErrorInvalidValue;
    });
}

}  // namespace a2t
