// Causal attention of a step's rows for fp32 caches (gfx950): chunks and decode (but for decode
// launches with one query head per KV head where attn_valu is the faster one).
//
//   attn_f32  one workgroup = (key split, QB blocks of 16 query rows, KV head,
//             stream), 8 waves: wave w takes every eighth 16-key block of the split;
//             the eight states are combined in LDS at the end.  With new rows in
//             the input it also rotates and stores them (fused append).
//
// fp32 products run on v_mfma_f32_16x16x4_f32 (fp32 inputs and sums at twice the vector
// ALU's rate without packed instructions), so that K and V are read once for 16 query rows
// and no product needs a cross-lane sum.  A lane's 16-byte reads are the A operands of four
// products each: the order of the contracted dims (scores) and of the output rows (values)
// is free.  V operands come straight from global memory; K goes through a region of LDS of
// the wave's own, because 16 lanes of a score operand are 16 rows: loaded directly they were
// 64 cache accesses per wave load instead of 16 (one query block: 43 against 31 us below).
// Nothing is shared between waves before the end, so there are no barriers in the loop, and
// the next block's K and V are in flight while one is computed.
//
// Measured (2 streams of ~2,100 keys and 22 rows, 32/8 heads of 128, 1.7 GFLOP of products
// with padding, 34 MB of K and V): a 4-layer step 896 -> 146 us, 27-28 us of it each layer's
// attention with the matrix units busy 30 % of the time and 35 MB read, where the vector ALU kernel (one workgroup per query row, 16 lanes per key)
// took 205 and the separate append 4.8; the products alone are 11 us and the bytes 6.  With 4
// waves, with every load of a block waited for at once, or with two workgroups per CU it was
// no faster.
//
// Order of the sums: a product adds its four terms and the running sum one after the other,
// so a sum that runs through many products rounds more often than the vector kernel's trees
// did.  Scores are summed in 16 parts, a block's P.V on its own, the waves' states in a
// tree: the error against 64 bits is the vector kernel's or less (2.0e-7 of 2.0e-7 there,
// 1.5e-7 of 1.6e-7 at 280 keys and head dim 64); with one sum each it was 2.5e-7 and 1.9e-7, and
// 6 % less time.
#include "a2t_internal.h"
#include "device_common.h"

#include <hip/hip_ext.h>
#include <math.h>

#include <type_traits>

namespace a2t {
namespace {

constexpr int kKeyBlock = 16;                        // keys (and query rows) of a product
constexpr int kKeyWaves = 8;     // waves of a workgroup: they share its keys

// 16 bytes of global memory (a pointer picked by branches would be loaded from as a flat
// address, and every flat load waits for all loads before it)
__device__ __forceinline__ f32x4 gload(const float* p) {
    return *reinterpret_cast<const __attribute__((address_space(1))) f32x4*>(reinterpret_cast<uintptr_t>(p));
}

// LDS accesses of the wave before this one come before those after it, whatever the compiler
// knows about their addresses in one lane (the hardware keeps a wave's LDS accesses in order)
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// max / sum over the four lanes l % 16 + 16 i that hold one query column
__device__ __forceinline__ float col_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float col_sum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Lane l of a wave is (query column l % 16, group lg = l / 16).
//   scores   S^T[16 keys x 16 queries]: A = K; product (s, j) contracts dims
//            16 s + 4 lg + j, so a lane needs K of key l % 16 at 16 s + 4 lg .. + 3;
//            the lane gets keys 4 lg + e, e < 4, of its query.
//   values   O^T[16 dims x 16 queries]: B = probabilities of key 4 lg + r (already
//            in the lane), A = V of key 4 lg + r; row i of product (b, j) is dim
//            64 b + 4 i + j, so a lane needs V at 64 b + 4 (l % 16) .. + 3; it gets
//            dims 64 b + 16 lg + 4 e + j.
template <int D, int QB, int N>
__global__ __launch_bounds__(64 * kKeyWaves, 2) void attn_f32_kernel(DevState st, AttnBatchT<N> b, WgStart<N> start,
                                                                     const float* q, float* o, const float* k_in,
                                                                     const float* v_in) {
    constexpr int KS = D / 16;   // 16-byte K loads of a lane per key block
    constexpr int NB = D / 64;   // 16-byte V loads of a lane per key
    constexpr int kScoreSums = 4;
    constexpr int CPR = D / 4;   // 16-byte chunks per row
    constexpr int kStride = kKeyWaves * kKeyBlock;
    constexpr int kExtra = QB == 1 ? KS * 64 : 0;
    __shared__ f32x4 s_mem[QB * kKeyWaves * 4 * NB * 64 + kExtra];
    f32x4(&s_part)[QB][kKeyWaves][4 * NB][64] = *reinterpret_cast<f32x4(*)[QB][kKeyWaves][4 * NB][64]>(s_mem);
    __shared__ float2 s_ml[QB][kKeyWaves][16];
    // the partial sums' place holds the Q operand and each wave's K block until the keys are done
    f32x4(&s_q)[QB][KS][64] = *reinterpret_cast<f32x4(*)[QB][KS][64]>(s_mem);
    f32x4* const s_k = s_mem + QB * KS * 64 + (threadIdx.x >> 6) * (kKeyBlock * CPR);
    static_assert(QB * KS * 64 + kKeyWaves * kKeyBlock * CPR <= QB * kKeyWaves * 4 * NB * 64 + kExtra, "they fit");

    int wg;
    const AttnDesc d = b.d[stream_of(start, b.count, &wg)];
    const int G = st.G, M = G * d.n_q, R = d.R;
    const int blocks = (M + kKeyBlock - 1) / kKeyBlock, groups = (blocks + QB - 1) / QB;
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };   // divisions run on the vector ALU
    // linear block (split, query group, KV head), heads fastest: the workgroups of a head
    // share an XCD's L2 when the head count divides the 8 XCDs
    const int y = uniform(wg / st.Hkv), g = wg - y * st.Hkv;
    const int sp = uniform(y / groups), grp = groups - 1 - (y - sp * groups);
    if (sp >= d.splits) return;
    const int w = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int mw = grp * QB * kKeyBlock;   // the workgroup's first query row
    const int vis0 = R - d.n_q;
    const int newbase = R - d.n_new;       // rows newbase .. R-1 come from k_in / v_in
    int qi[QB], hh[QB];                    // row and head of the lane's queries (past M: row M-1)
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        const int mqc = min(mw + x * kKeyBlock + l16, M - 1);
        qi[x] = mqc / G;
        hh[x] = mqc - qi[x] * G;
    }
    // the last group sees every key: it stores the new rows
    const bool writer = d.n_new > 0 && grp == groups - 1;
    const int last_i = uniform((min(M, mw + QB * kKeyBlock) - 1) / G);
    const int k_end = vis0 + last_i + 1;
    const int t0 = sp * d.tile_q + min(sp, d.tile_r), t1 = t0 + d.tile_q + (sp < d.tile_r ? 1 : 0);
    // this wave's key blocks: k0, k0 + kStride, ..; n of them
    const int k0 = t0 * kTileKeys + w * kKeyBlock;
    const int n = max(0, (min(k_end, t1 * kTileKeys) - k0 + kStride - 1) / kStride);

    const int kept = d.kept, head = d.head, ring_rows = st.unit_rows;
    const float* kk = static_cast<const float*>(st.k_kept) + pool_index(st, b.layer, d.s, g, st.kept_rows, 0);
    const float* vk = static_cast<const float*>(st.v_kept) + pool_index(st, b.layer, d.s, g, st.kept_rows, 0);
    float* ku = static_cast<float*>(st.k_unit) + pool_index(st, b.layer, d.s, g, ring_rows, 0);
    float* vu = static_cast<float*>(st.v_unit) + pool_index(st, b.layer, d.s, g, ring_rows, 0);
    auto ring_slot = [&](int j) {
        const int slot = head + (j - kept);
        return slot >= ring_rows ? slot - ring_rows : slot;
    };
    auto row = [&](const float* reg_kept, const float* reg_ring, const float* in, int j) -> const float* {
        j = min(j, R - 1);   // keys past R read row R-1 and are masked
        if (j >= newbase) return in + ((int64_t)(d.in_row0 + (j - newbase)) * st.Hkv + g) * D;
        return j < kept ? reg_kept + (int64_t)j * D : reg_ring + (int64_t)ring_slot(j) * D;
    };

    f32x4 acc[QB][NB][4];
    float mrun[QB], lrun[QB];
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        mrun[x] = -INFINITY;
        lrun[x] = 0.f;
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[x][c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // element offsets of a key block's rows from the ring when the block is one run of
    // resident rows
    const int64_t to_kept = (static_cast<const float*>(st.k_kept) - static_cast<const float*>(st.k_unit)) +
                            pool_index(st, b.layer, d.s, g, st.kept_rows, 0) - pool_index(st, b.layer, d.s, g, ring_rows, 0);
    auto run_of = [&](int kb, int64_t* off) {
        if (kb + kKeyBlock > newbase) return false;
        if (kb + kKeyBlock <= kept) {
            *off = to_kept + (int64_t)kb * D;
            return true;
        }
        const int slot = ring_slot(kb);
        *off = (int64_t)slot * D;
        return kb >= kept && slot + kKeyBlock <= ring_rows;
    };
    f32x4 kc[KS], vc[4][NB];
    // K of a block, whole rows at a time (the 16 rows of an operand would be 16 cache lines
    // per quarter of a wave's load), through LDS into the operands' order
    auto load_k = [&](int kb, int ln) {
        int64_t off;
        if (run_of(kb, &off)) {
            const float* p = ku + off + 4 * ln;
#pragma unroll
            for (int i = 0; i < KS; ++i) kc[i] = gload(p + 256 * i);
        } else {
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                kc[i] = gload(row(kk, ku, k_in, kb + (64 * i + ln) / CPR) + 4 * (ln % CPR));
                asm volatile("" ::: "memory");   // one row's address at a time (registers)
            }
        }
    };
    // chunk c of key r of the wave's block: swizzled, so that neither the rows nor the
    // 16 keys of one chunk have a bank conflict
    auto k_at = [&](int r, int c) -> f32x4& { return s_k[r * CPR + (c ^ r)]; };
    auto load_v = [&](int kb, int ln) {
        int64_t off;
        if (run_of(kb, &off)) {
            const float* p = vu + off + (4 * (ln >> 4)) * D + 4 * (ln & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < NB; ++c) vc[r][c] = gload(p + r * D + 64 * c);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float* p = row(vk, vu, v_in, kb + 4 * (ln >> 4) + r) + 4 * (ln & 15);
#pragma unroll
                for (int c = 0; c < NB; ++c) vc[r][c] = gload(p + 64 * c);
                asm volatile("" ::: "memory");   // one row's address at a time (registers)
            }
        }
    };
    if (n > 0) {
        load_k(k0, lane);
        load_v(k0, lane);
    }
    // Q^T operand of the query blocks, rotated and scaled by scale * log2(e), in LDS: each
    // of the first waves does a part.  Rows past M read row M - 1 and are never stored.
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        const float* qp = q + ((int64_t)(d.q_row0 + qi[x]) * st.Hq + g * G + hh[x]) * D + 4 * lg;
        const float2* cp = st.rope + ((int64_t)d.s * st.max_step_rows + d.rope_row0 + qi[x]) * (D / 2) + 4 * lg;
        for (int s = w; s < KS / 2; s += kKeyWaves) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(qp + 16 * s);
            const f32x4 a2 = *reinterpret_cast<const f32x4*>(qp + 16 * s + D / 2);
            const float4 c01 = *reinterpret_cast<const float4*>(cp + 16 * s);
            const float4 c23 = *reinterpret_cast<const float4*>(cp + 16 * s + 2);
            const float cs[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
            f32x4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo[j] = (a[j] * cs[j] - a2[j] * sn[j]) * st.scale_log2e;
                hi[j] = (a2[j] * cs[j] + a[j] * sn[j]) * st.scale_log2e;
            }
            s_q[x][s][lane] = lo;
            s_q[x][s + KS / 2][lane] = hi;
        }
    }
    __syncthreads();

    if (n > 0) {
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
            const int kb = k0 + i * kStride;
            // registers: the Q operand is read from LDS in every pass, and no address of the
            // lane is kept from one pass to the next
            int ln = lane;
            asm volatile("" : "+v"(ln)::"memory");
            const int l16 = ln & 15, lg = ln >> 4;
#pragma unroll
            for (int i2 = 0; i2 < KS; ++i2) k_at((64 * i2 + ln) / CPR, ln % CPR) = kc[i2];
            wave_lds_order();   // other lanes read these rows
            if (i + 1 < n) load_k(kb + kStride, ln);
            if (d.n_new > 0 && kb + kKeyBlock > newbase) {
                // rotate the keys that are new (the rotate-half partner of a lane's chunk s
                // is its own chunk s + KS / 2) and store their rows
                const int j = min(kb + l16, R - 1);
                const bool is_new = j >= newbase;
                const float2* cp = st.rope + ((int64_t)d.s * st.max_step_rows + max(j - newbase, 0)) * (D / 2) + 4 * lg;
                float* const p = is_new && kb + l16 < R && writer ? ku + (int64_t)ring_slot(j) * D + 4 * lg : nullptr;
#pragma unroll
                for (int s = 0; s < KS / 2; ++s) {
                    const float4 c01 = *reinterpret_cast<const float4*>(cp + 16 * s);
                    const float4 c23 = *reinterpret_cast<const float4*>(cp + 16 * s + 2);
                    const float cs[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
                    const f32x4 a = k_at(l16, 4 * s + lg), a2 = k_at(l16, 4 * s + lg + CPR / 2);
                    f32x4 lo, hi;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        lo[e] = a[e] * cs[e] - a2[e] * sn[e];
                        hi[e] = a2[e] * cs[e] + a[e] * sn[e];
                    }
                    if (is_new) {
                        k_at(l16, 4 * s + lg) = lo;
                        k_at(l16, 4 * s + lg + CPR / 2) = hi;
                    }
                    if (p) {
                        *reinterpret_cast<f32x4*>(p + 16 * s) = lo;
                        *reinterpret_cast<f32x4*>(p + 16 * s + D / 2) = hi;
                    }
                }
                if (writer) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int jv = kb + 4 * lg + r;
                        if (jv >= newbase && jv < R) {
                            float* p = vu + (int64_t)ring_slot(jv) * D + 4 * l16;
#pragma unroll
                            for (int c = 0; c < NB; ++c) *reinterpret_cast<f32x4*>(p + 64 * c) = vc[r][c];
                        }
                    }
                }
                // nothing of this path in flight past it: the loads of the loop's own order are
                // then waited for one group at a time
                wait_vmem<0>();
            }
            // scores: sums of D / 16 products, then a tree of them (the products add one after
            // the other in a sum)
            f32x4 sc[QB];
#pragma unroll
            for (int x = 0; x < QB; ++x) {
                f32x4 sum[kScoreSums];
#pragma unroll
                for (int u = 0; u < kScoreSums; ++u) {
                    f32x4 s4[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) s4[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = u * KS / kScoreSums; s < (u + 1) * KS / kScoreSums; ++s) {
                        const f32x4 kv = k_at(l16, 4 * s + lg), qv = s_q[x][s][ln];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            s4[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j], qv[j], s4[j], 0, 0, 0);
                    }
                    sum[u] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
                }
                sc[x] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
                asm volatile("" ::: "memory");   // K is read again for the next query block: registers
            }
            const bool masked = kb + kKeyBlock - 1 > vis0;
            float p[QB][4];
#pragma unroll
            for (int x = 0; x < QB; ++x) {
                if (masked) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (kb + 4 * lg + e > vis0 + qi[x]) sc[x][e] = -INFINITY;
                }
                const float tmax = col_max(fmaxf(fmaxf(sc[x][0], sc[x][1]), fmaxf(sc[x][2], sc[x][3])));
                // the reference follows the row maximum lazily: raised (and the running sums
                // rescaled) only when a block exceeds it by more than 2^8
                if (__any(tmax > mrun[x] + 8.f)) {
                    const float mn = fmaxf(mrun[x], tmax);
                    const float corr = __builtin_amdgcn_exp2f(mrun[x] - ((mn == -INFINITY) ? 0.f : mn));
                    lrun[x] *= corr;
#pragma unroll
                    for (int c = 0; c < NB; ++c)
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[x][c][j] *= corr;
                    mrun[x] = mn;
                }
                const float mu = (mrun[x] == -INFINITY) ? 0.f : mrun[x];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[x][e] = __builtin_amdgcn_exp2f(sc[x][e] - mu);
                lrun[x] += (p[x][0] + p[x][1]) + (p[x][2] + p[x][3]);
            }
            // a masked key has probability 0, which would still turn an infinite or NaN value
            // of it into NaN: blocks that hold both take the vector ALU, key by key
            bool plain = true;
            if (masked) {
                float z = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < NB; ++c)
#pragma unroll
                        for (int e = 0; e < 4; ++e) z = fmaf(vc[r][c][e], 0.f, z);
                plain = !__any(z != 0.f);   // inf * 0 and NaN * 0 are NaN
            }
            if (plain) {
                // a block's products are summed on their own: the running sums of a long split
                // would otherwise round once per product
#pragma unroll
                for (int x = 0; x < QB; ++x)
#pragma unroll
                    for (int c = 0; c < NB; ++c) {
                        f32x4 sum[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) sum[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                sum[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[r][c][j], p[x][r], sum[j], 0, 0, 0);
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[x][c][j] += sum[j];
                    }
            } else {
#pragma unroll 1
                for (int k4 = 0; k4 < kKeyBlock; k4 += 4) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float* pv = row(vk, vu, v_in, kb + k4 + r) + 16 * lg;
#pragma unroll
                        for (int x = 0; x < QB; ++x) {
                            const float px = __shfl(p[x][r], l16 + 4 * k4);
                            if (kb + k4 + r > vis0 + qi[x]) continue;
#pragma unroll
                            for (int c = 0; c < NB; ++c)
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const f32x4 v = gload(pv + 64 * c + 4 * e);
#pragma unroll
                                    for (int j = 0; j < 4; ++j) acc[x][c][j][e] = fmaf(px, v[j], acc[x][c][j][e]);
                                    asm volatile("" ::: "memory");   // one load at a time (registers)
                                }
                        }
                    }
                }
            }
            if (i + 1 < n) load_v(kb + kStride, ln);
        }
#pragma unroll
        for (int x = 0; x < QB; ++x) lrun[x] = col_sum(lrun[x]);
    }
    __syncthreads();   // the Q operand's place takes the sums

    // combine the waves' states: each wave sums an eighth of the dims
#pragma unroll
    for (int x = 0; x < QB; ++x) {
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s_part[x][w][4 * c + e][lane] = f32x4{acc[x][c][0][e], acc[x][c][1][e], acc[x][c][2][e], acc[x][c][3][e]};
        if (lg == 0) s_ml[x][w][l16] = make_float2(mrun[x], lrun[x]);
    }
    __syncthreads();
    const bool whole = d.splits == 1;
    float* po = st.ws + d.ws_off;
#pragma unroll
    for (int x = 0; x < QB; ++x) {
        const int mq = mw + x * kKeyBlock + l16;
        if (mq >= M) return;
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < kKeyWaves; ++k) mx = fmaxf(mx, s_ml[x][k][l16].x);
        auto weight = [&](int k) {
            const float m = s_ml[x][k][l16].x;
            return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
        };
        auto tree = [](auto&& f) { return ((f(0) + f(1)) + (f(2) + f(3))) + ((f(4) + f(5)) + (f(6) + f(7))); };
        static_assert(kKeyWaves == 8, "the tree's leaves");
        const float L = tree([&](int k) { return weight(k) * s_ml[x][k][l16].y; });
        const int64_t at = ((int64_t)sp * st.Hkv + g) * M + mq;
        float* orow = whole ? o + ((int64_t)(d.q_row0 + qi[x]) * st.Hq + g * G + hh[x]) * D : po + at * D;
        for (int pi = w; pi < 4 * NB; pi += kKeyWaves) {   // dims 64 (pi / 4) + 16 lg + 4 (pi % 4) .. + 3
            f32x4 O = tree([&](int k) { return s_part[x][k][pi][lane] * weight(k); });
            if (whole) {
#pragma unroll
                for (int j = 0; j < 4; ++j) O[j] /= L;
            }
            *reinterpret_cast<f32x4*>(orow + 64 * (pi >> 2) + 16 * lg + 4 * (pi & 3)) = O;
        }
        if (!whole && w == 0 && lg == 0)
            *reinterpret_cast<float2*>(po + (int64_t)d.splits * st.Hkv * M * D + at * 2) = make_float2(mx, L);
    }
}

}  // namespace

hipError_t launch_attn_f32(const DevState& st, const AttnBatch& b, int query_blocks, const void* q, void* o,
                           const void* k_in, const void* v_in, hipStream_t stream, const KTimer& kt) {
    const dim3 block(64 * kKeyWaves);
    const float *qq = static_cast<const float*>(q), *ki = static_cast<const float*>(k_in), *vi = static_cast<const float*>(v_in);
    float* oo = static_cast<float*>(o);
    return by_size<AttnBatchT>(b, [&](const auto& bb) {
        constexpr int N = sizeof(bb.d) / sizeof(bb.d[0]);
        WgStart<N> start{};
        const dim3 grid = place_workgroups(b.count, &start, [&](int i) {
            return f32_groups(st.G * b.d[i].n_q, query_blocks) * b.d[i].splits * st.Hkv;
        });
        auto go = [&](auto kernel) {
            if (kt.start)
                hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, kt.start, kt.stop, 0, st, bb, start, qq, oo, ki, vi);
            else
                hipLaunchKernelGGL(kernel, grid, block, 0, stream, st, bb, start, qq, oo, ki, vi);
            return hipGetLastError();
        };
        if (st.D == 128) return query_blocks == 1 ? go(attn_f32_kernel<128, 1, N>) : go(attn_f32_kernel<128, 2, N>);
        if (st.D == 64) return query_blocks == 1 ? go(attn_f32_kernel<64, 1, N>) : go(attn_f32_kernel<64, 2, N>);
        return hipErrorInvalidValue;
    });
}

}  // namespace a2t
