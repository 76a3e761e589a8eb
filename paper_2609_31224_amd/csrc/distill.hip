// The adaptation objective of Sec. 3.2 on given logits: masked cross-entropy
// over transcription rows, T^2 KL(P_T || P_S) at native rows with the teacher
// extended by zero probability on the added tokens, group-balanced means, and
// the gradient with respect to the student logits.  Public API: include/a2t.h.
//
//   distill_row_kernel     one workgroup per row, sized so that its threads hold
//                          the whole student row in registers (as it is stored,
//                          16 bytes a chunk): every load is in flight at once and
//                          the gradient needs no second read.  Transcription rows
//                          read the student only: (max, sum 2^x) of s log2 e.
//                          Native rows stream the teacher beside it: the same
//                          pair for s/T and t/T, and A = sum_v p_v (t_v - s_v) / T,
//                          which gives KL = A / Z_w - lse(w) + lse(u) in the same
//                          pass (u = s/T, w = t/T); the first chunks of the
//                          teacher stay in LDS for the gradient, the rest is read
//                          again.
//   distill_reduce_kernel  one workgroup: the four weighted sums over rows in
//                          a fixed order (deterministic).
// The weights of the four means are per-row coefficients computed on the host
// from the row metadata.
#include "../../include/a2t.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

namespace {

constexpr int kReduceThreads = 256;
constexpr int kRowThreads = 1024;   // most threads of a row's workgroup
constexpr int kChunk = 8;           // elements per chunk (16 bytes of bf16, 32 of fp32)
constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kLn2 = 0.693147180559945309417f;

// Chunks of its row a thread holds in registers: 76 (bf16) or 72 (fp32) of the 128
// registers that a thread of a full CU (16 waves) has, so a row of up to 155,648
// (73,728) logits is read once; chunks of the teacher it keeps in LDS, 128 bytes per
// thread, 128 KiB for a CU's 1,024 threads; and chunks of the teacher it requests
// ahead of the one it works on.
template <typename T> struct Hold;

// 20 bytes: a table of up to 16 KiB is copied by the runtime ~10 us faster than a larger one
// (739 rows of 24 bytes: 18.6 -> 30.6 us a pass).
struct DistillRow {
    int32_t row;        // row of the batch (rows are dispatched costliest first)
    int32_t target;     // ASR target, -1 elsewhere
    float c_main;       // weight of this row's CE in L_ASR (target >= 0), else of its KL in L_native
    float c_dec;        // ... in L_dec
    float c_turn;       // ... in L_turn
};
static_assert(sizeof(DistillRow) == 20, "rows of the table");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct bf16_t {
    uint16_t bits;
};

// one chunk as stored
template <typename T> struct Raw;
template <> struct Raw<bf16_t> {
    u32x4 a;
};
template <> struct Raw<float> {
    u32x4 a, b;
};
template <> struct Hold<bf16_t> {
    static constexpr int kRegs = 19, kLds = 8, kAhead = 3;
};
template <> struct Hold<float> {
    static constexpr int kRegs = 9, kLds = 4, kAhead = 1;
};
// chunk c of a row (a scalar base and a 32-bit offset: rows stay under 4 GiB)
__device__ __forceinline__ Raw<bf16_t> load_raw(const bf16_t* row, int c) {
    return {*reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(row) + (uint32_t)c * 16u)};
}
__device__ __forceinline__ Raw<float> load_raw(const float* row, int c) {
    const u32x4* p = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(row) + (uint32_t)c * 32u);
    return {p[0], p[1]};
}
// How a bf16 pair comes apart, as values the compiler knows nothing about: each sweep
// over the held chunks takes its own, so that none of the 152 logits a thread unpacks
// is kept for the next sweep in a register of its own.
struct Apart {
    uint32_t shift, mask;
    __device__ __forceinline__ Apart() {
        asm volatile("s_mov_b32 %0, 16" : "=s"(shift));
        asm volatile("s_mov_b32 %0, 0xffff0000" : "=s"(mask));
    }
};
__device__ __forceinline__ void unpack(const Raw<bf16_t>& r, const Apart& ap, float (&x)[kChunk]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[2 * e] = __uint_as_float(r.a[e] << ap.shift);
        x[2 * e + 1] = __uint_as_float(r.a[e] & ap.mask);
    }
}
__device__ __forceinline__ void unpack(const Raw<float>& r, const Apart&, float (&x)[kChunk]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = __uint_as_float(r.a[e]);
        x[4 + e] = __uint_as_float(r.b[e]);
    }
}
// elements from `first` on become -inf
__device__ __forceinline__ void cut(Raw<bf16_t>& r, int first) {
    uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (2 * e >= first) w[e] = (w[e] & 0xffff0000u) | 0xff80u;
        if (2 * e + 1 >= first) w[e] = (w[e] & 0x0000ffffu) | 0xff800000u;
    }
    r.a = u32x4{w[0], w[1], w[2], w[3]};
}
__device__ __forceinline__ void cut(Raw<float>& r, int first) {
    uint32_t w[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (e >= first) w[e] = 0xff800000u;
    r.a = u32x4{w[0], w[1], w[2], w[3]};
    r.b = u32x4{w[4], w[5], w[6], w[7]};
}
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const bf16_t* p) { return __uint_as_float((uint32_t)p->bits << 16); }

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    const bf16x2 v = {(__bf16)a, (__bf16)b};   // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ void store_chunk(float* row, int c, const float (&g)[kChunk]) {
    float4* p = reinterpret_cast<float4*>(reinterpret_cast<char*>(row) + (uint32_t)c * 32u);
    p[0] = make_float4(g[0], g[1], g[2], g[3]);
    p[1] = make_float4(g[4], g[5], g[6], g[7]);
}
// A bf16 gradient goes out in whole cache lines, to be read by a later kernel from
// more rows than L2 holds: non-temporal stores do not displace the logits (237 -> 228
// us, below).  An fp32 chunk is two stores of half lines: 199 us ordinary, 214 us
// non-temporal on 1,000 rows of 80,002 logits.
__device__ __forceinline__ void store_chunk(bf16_t* row, int c, const float (&g)[kChunk]) {
    __builtin_nontemporal_store(u32x4{pack2(g[0], g[1]), pack2(g[2], g[3]), pack2(g[4], g[5]), pack2(g[6], g[7])},
                                reinterpret_cast<u32x4*>(reinterpret_cast<char*>(row) + (uint32_t)c * 16u));
}

// Running sums in the log2 domain: z = sum 2^(k x - m) with m at least the largest
// k x so far, rounded.  m is the reference exactly as it was subtracted, so log2 of the
// whole sum is m + log2 z with no error from rounding k x.  The rounding moves the
// exponents by up to ulp(m) / 2, which is nothing at kFar (2^-5) and would overflow at
// 2^32: m starts at -kFar, below which a logit counts as 0 beside any other (masks of
// -1e30 or of the type's lowest value), and a row whose m ends up at kFar or further
// out is computed again from exact differences (the kernel's end).
constexpr float kFar = 1048576.f;
struct Sum {
    float m, z;
};
// the teacher's, with a = sum 2^(k t - m) (t - s)
struct SumA {
    float m, z, a;
};
__device__ __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }

// largest logit of a chunk, and of mx
template <typename T>
__device__ __forceinline__ float max_of(const Raw<T>& r, const Apart& ap, float mx) {
    float x[kChunk];
    unpack(r, ap, x);
#pragma unroll
    for (int e = 0; e < kChunk; ++e) mx = fmaxf(mx, x[e]);
    return mx;
}
// raises the reference to the largest logit mx of the chunks about to be added
__device__ __forceinline__ void raise(Sum& s, float mx, float k) {
    const float mn = fmaxf(s.m, mx * k);
    s.z *= exp2_(s.m - mn);
    s.m = mn;
}
__device__ __forceinline__ void raise(SumA& w, float mx, float k) {
    const float mn = fmaxf(w.m, mx * k), sc = exp2_(w.m - mn);
    w.z *= sc;
    w.a *= sc;
    w.m = mn;
}
// adds a chunk of the student
template <typename T>
__device__ __forceinline__ void add(Sum& s, const Raw<T>& r, const Apart& ap, float k) {
    float x[kChunk], z = 0.f;
    unpack(r, ap, x);
#pragma unroll
    for (int e = 0; e < kChunk; ++e) z += exp2_(fmaf(x[e], k, -s.m));
    s.z += z;
}
// adds a chunk of the teacher t beside the student s
template <typename T>
__device__ __forceinline__ void add(SumA& w, const Raw<T>& t, const Raw<T>& s, const Apart& ap, float k) {
    float x[kChunk], y[kChunk], z = 0.f, a = 0.f;
    unpack(t, ap, x);
    unpack(s, ap, y);
#pragma unroll
    for (int e = 0; e < kChunk; ++e) {
        const float p = exp2_(fmaf(x[e], k, -w.m));
        z += p;
        // a token the teacher rules out (and the added ones) contributes nothing
        a += x[e] == -INFINITY ? 0.f : p * (x[e] - y[e]);
    }
    w.z += z;
    w.a += a;
}
__device__ __forceinline__ void merge(Sum& x, const Sum& y) {
    const float mn = fmaxf(x.m, y.m);
    x.z = x.z * exp2_(x.m - mn) + y.z * exp2_(y.m - mn);
    x.m = mn;
}
__device__ __forceinline__ void merge(SumA& x, const SumA& y) {
    const float mn = fmaxf(x.m, y.m);
    const float cx = exp2_(x.m - mn), cy = exp2_(y.m - mn);
    x.z = x.z * cx + y.z * cy;
    x.a = x.a * cx + y.a * cy;
    x.m = mn;
}
// over the workgroup: waves by xor shuffles, then across waves in LDS; every thread
// returns the same sums (one barrier inside)
__device__ __forceinline__ void reduce(Sum& u, SumA* w, float* part) {
#pragma unroll
    for (int mask = 32; mask >= 1; mask >>= 1) {
        merge(u, Sum{__shfl_xor(u.m, mask), __shfl_xor(u.z, mask)});
        if (w) merge(*w, SumA{__shfl_xor(w->m, mask), __shfl_xor(w->z, mask), __shfl_xor(w->a, mask)});
    }
    const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        float* p = part + 5 * wave;
        p[0] = u.m, p[1] = u.z;
        if (w) p[2] = w->m, p[3] = w->z, p[4] = w->a;
    }
    __syncthreads();
    u = Sum{part[0], part[1]};
    if (w) *w = SumA{part[2], part[3], part[4]};
    for (int x = 1; x < waves; ++x) {
        const float* p = part + 5 * x;
        merge(u, Sum{p[0], p[1]});
        if (w) merge(*w, SumA{p[2], p[3], p[4]});
    }
}

// chunks are worked through one group after the other: no more of them are unpacked at once
__device__ __forceinline__ void in_turn() { __builtin_amdgcn_sched_barrier(0); }

// grid: one workgroup per row.  Bound: HBM, once the row is read and its gradient
// written one time each; per logit a transcription row costs ~8 vector operations and
// two exponentials, a native row about twice that.  Measured on 1,340 rows of 151,938
// bf16 logits (957 of them transcription rows), with gradient: 228 us, 4.1 TB/s (480 us
// with one 256-thread workgroup per row that kept online maxima per chunk, read the
// teacher of every row and read both again for the gradient: bound by ~75 vector
// operations per logit); teacher re-read whole instead of from LDS: 231 us.
template <typename T, bool GRAD, int NR>
__global__ __launch_bounds__(kRowThreads) void distill_row_kernel(
    const T* student, int64_t s_stride, const T* teacher, int64_t t_stride, int vocab, int vs,
    const DistillRow* rows, float inv_t, float2* rowval, T* grad) {
    constexpr int NL = NR < Hold<T>::kLds ? NR : Hold<T>::kLds;
    extern __shared__ u32x4 t_lds[];           // GRAD: NL chunks of the teacher per thread
    __shared__ float part[5 * kRowThreads / 64];
    const int tid = threadIdx.x, TH = blockDim.x;
    const DistillRow r = rows[blockIdx.x];
    const T* s = student + (int64_t)r.row * s_stride;
    const T* t = teacher + (int64_t)r.row * t_stride;
    T* g = GRAD ? grad + (int64_t)r.row * s_stride : nullptr;
    const float wk = r.target < 0 ? r.c_main + r.c_dec + r.c_turn : 0.f;   // KL weight in the gradient
    const float wc = r.target < 0 ? 0.f : r.c_main;                        // CE weight in the gradient
    const int nc = (vs + kChunk - 1) / kChunk, nt = (vocab + kChunk - 1) / kChunk;   // chunks

    if (wk == 0.f && wc == 0.f) {  // a row without loss: zero gradient
        const float z[kChunk] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (GRAD)
            for (int c = tid; c < nc; c += TH) store_chunk(g, c, z);
        if (tid == 0) rowval[blockIdx.x] = make_float2(0.f, 0.f);
        return;
    }

    // the thread's chunk of round k, computed where it is used and not kept
    auto chunk_no = [&](int k) {
        int x = tid;
        asm volatile("" : "+v"(x));
        return k * TH + x;
    };
    // chunk c of the student (teacher), -inf past its last logit; the address is clamped
    // so that the loads need no branch
    auto student_chunk = [&](int c) { return load_raw(s, min(c, nc - 1)); };
    auto teacher_chunk = [&](int c) { return load_raw(t, min(c, nt - 1)); };
    // c0: the first chunk of the workgroup's round that holds chunk c
    auto cut_student = [&](Raw<T>& x, int c, int c0) {
        if ((c0 + TH) * kChunk > vs) cut(x, vs - c * kChunk);
    };
    auto cut_teacher = [&](Raw<T>& x, int c, int c0) {
        if ((c0 + TH) * kChunk > vocab) cut(x, vocab - c * kChunk);
    };

    Raw<T> hs[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) hs[k] = student_chunk(chunk_no(k));
    const float target_logit = wc != 0.f && tid == 0 ? load1(s + r.target) : 0.f;
#pragma unroll
    for (int k = 0; k < NR; ++k) cut_student(hs[k], chunk_no(k), k * TH);

    const Apart to_max, to_sum;
    const bool native = wk != 0.f;
    const float kt = inv_t * kLog2e, tt = 1.f / inv_t;
    if (!native) {
        // ---- transcription row: the student at temperature 1
        constexpr float k1 = kLog2e;
        Sum u{-kFar, 0.f};
#pragma unroll
        for (int k = 0; k < NR; k += 4) {   // in groups of four chunks
            constexpr int N = 4;
            float mx = -INFINITY;
            if (k * TH < nc) {
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (k + e < NR) mx = max_of(hs[k + e], to_max, mx);
            }
            if (k * TH < nc) {
                raise(u, mx, k1);
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (k + e < NR) add(u, hs[k + e], to_sum, k1);
            }
            in_turn();
        }
        for (int c = NR * TH + tid; c - tid < nc; c += TH) {
            Raw<T> x = student_chunk(c);
            cut_student(x, c, c - tid);
            raise(u, max_of(x, to_max, -INFINITY), k1);
            add(u, x, to_sum, k1);
        }
        reduce(u, nullptr, part);
        if (fabsf(u.m) < kFar) {
            if (tid == 0) rowval[blockIdx.x] = make_float2(kLn2 * (u.m + __builtin_amdgcn_logf(u.z)) - target_logit, 0.f);
            if (!GRAD) return;
            // dL/ds_v = wc (softmax(s)_v - [v == target])
            const float coef = wc / u.z;
            const Apart to_write;
            auto write = [&](const Raw<T>& x, int c) {
                float y[kChunk];
                unpack(x, to_write, y);
#pragma unroll
                for (int e = 0; e < kChunk; ++e) y[e] = coef * exp2_(fmaf(y[e], k1, -u.m));
                if (c == r.target / kChunk) {
#pragma unroll
                    for (int e = 0; e < kChunk; ++e) y[e] -= e == r.target % kChunk ? wc : 0.f;
                }
                if (c < nc) store_chunk(g, c, y);
            };
#pragma unroll
            for (int k = 0; k < NR; ++k)
            {
                if (k * TH < nc) write(hs[k], chunk_no(k));
                in_turn();
            }
            for (int c = NR * TH + tid; c - tid < nc; c += TH) {
                Raw<T> x = student_chunk(c);
                cut_student(x, c, c - tid);
                write(x, c);
            }
            return;
        }
    } else {
        // ---- native row: student and teacher at temperature T
        Sum u{-kFar, 0.f};
        SumA w{-kFar, 0.f, 0.f};
        constexpr int NA = NR - 1 < Hold<T>::kAhead ? NR - 1 : Hold<T>::kAhead;
        Raw<T> ts[NR];   // in flight: NA chunks ahead of the one in work
#pragma unroll
        for (int k = 0; k < NA; ++k) ts[k] = teacher_chunk(chunk_no(k));
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            if (k + NA < NR) ts[k + NA] = teacher_chunk(chunk_no(k + NA));
            const int c = chunk_no(k);
            Raw<T> x = ts[k];
            cut_teacher(x, c, k * TH);
            if (GRAD && k < NL) reinterpret_cast<Raw<T>*>(t_lds)[c] = x;
            float mu = -INFINITY, mw = -INFINITY;
            if (k * TH < nc) {
                mu = max_of(hs[k], to_max, mu);
                mw = max_of(x, to_max, mw);
            }
            if (k * TH < nc) {
                raise(u, mu, kt);
                add(u, hs[k], to_sum, kt);
                raise(w, mw, kt);
                add(w, x, hs[k], to_sum, kt);
            }
            in_turn();
        }
        for (int c = NR * TH + tid; c - tid < nc; c += TH) {
            Raw<T> x = student_chunk(c), y = teacher_chunk(c);
            cut_student(x, c, c - tid);
            cut_teacher(y, c, c - tid);
            raise(u, max_of(x, to_max, -INFINITY), kt);
            add(u, x, to_sum, kt);
            raise(w, max_of(y, to_max, -INFINITY), kt);
            add(w, y, x, to_sum, kt);
        }
        reduce(u, &w, part);
        if (fabsf(u.m) < kFar && fabsf(w.m) < kFar) {
            if (tid == 0) {
                const float lse = (u.m - w.m) + (__builtin_amdgcn_logf(u.z) - __builtin_amdgcn_logf(w.z));
                rowval[blockIdx.x] = make_float2(0.f, tt * tt * (inv_t * w.a / w.z + kLn2 * lse));
            }
            if (!GRAD) return;
            // dL/ds_v = wk T (softmax(u)_v - p_t,v)
            const float cu = wk * tt / u.z, cw = wk * tt / w.z;
            const Apart to_write;
            auto write = [&](const Raw<T>& x, const Raw<T>& y, int c) {
                float a[kChunk], b[kChunk];
                unpack(x, to_write, a);
                unpack(y, to_write, b);
#pragma unroll
                for (int e = 0; e < kChunk; ++e)
                    a[e] = cu * exp2_(fmaf(a[e], kt, -u.m)) - cw * exp2_(fmaf(b[e], kt, -w.m));
                if (c < nc) store_chunk(g, c, a);
            };
#pragma unroll
            for (int k = NL; k < NL + NA; ++k)
                if (k < NR) ts[k] = teacher_chunk(chunk_no(k));
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                // the chunks that LDS holds are written while the others are on their way
                if (k >= NL && k + NA < NR) ts[k + NA] = teacher_chunk(chunk_no(k + NA));
                if (k * TH < nc) {
                    const int c = chunk_no(k);
                    Raw<T> y;
                    if (k < NL) {
                        y = reinterpret_cast<const Raw<T>*>(t_lds)[c];   // written by this thread
                    } else {
                        y = ts[k];
                        cut_teacher(y, c, k * TH);
                    }
                    write(hs[k], y, c);
                }
                in_turn();
            }
            for (int c = NR * TH + tid; c - tid < nc; c += TH) {
                Raw<T> x = student_chunk(c), y = teacher_chunk(c);
                cut_student(x, c, c - tid);
                cut_teacher(y, c, c - tid);
                write(x, y, c);
            }
            return;
        }
    }

    // ---- a row with a largest k x of kFar or beyond, or none above -kFar: the largest logits
    // first, then sums of 2^(k (x - largest)), whose differences are exact or far below 0
    const T* const other = native ? t : s;   // a transcription row has no use for its second row
    const int others = native ? vocab : vs;
    auto each = [&](auto f) {
        for (int c = tid; c < nc; c += TH) {
            Raw<T> x = load_raw(s, c), y = load_raw(other, min(c, (others - 1) / kChunk));
            cut(x, vs - c * kChunk);
            cut(y, others - c * kChunk);
            float a[kChunk], b[kChunk];
            unpack(x, to_sum, a);
            unpack(y, to_sum, b);
            f(c, a, b);
        }
    };
    const float kx = native ? kt : kLog2e;
    float ms = -INFINITY, mt = -INFINITY, zs = 0.f, zt = 0.f, at = 0.f;
    each([&](int, const float(&a)[kChunk], const float(&b)[kChunk]) {
#pragma unroll
        for (int e = 0; e < kChunk; ++e) ms = fmaxf(ms, a[e]), mt = fmaxf(mt, b[e]);
    });
    const auto over_row = [&](float us, float uz, float wm, float wz, float wa, float (&out)[5]) {
        Sum u{us, uz};
        SumA w{wm, wz, wa};
        __syncthreads();
        reduce(u, &w, part);
        out[0] = u.m, out[1] = u.z, out[2] = w.m, out[3] = w.z, out[4] = w.a;
    };
    float all[5];
    over_row(ms, 0.f, mt, 0.f, 0.f, all);
    ms = all[0], mt = all[2];
    each([&](int, const float(&a)[kChunk], const float(&b)[kChunk]) {
#pragma unroll
        for (int e = 0; e < kChunk; ++e) {
            zs += exp2_((a[e] - ms) * kx);
            const float p = exp2_((b[e] - mt) * kx);
            zt += p;
            at += b[e] == -INFINITY ? 0.f : p * ((b[e] - a[e]) * inv_t);
        }
    });
    over_row(0.f, zs, 0.f, zt, at, all);
    zs = all[1], zt = all[3], at = all[4];
    const float lu = kLn2 * __builtin_amdgcn_logf(zs), lw = kLn2 * __builtin_amdgcn_logf(zt);
    if (tid == 0)
        rowval[blockIdx.x] = native ? make_float2(0.f, tt * tt * (at / zt + (ms - mt) * inv_t + (lu - lw)))
                                    : make_float2((ms - target_logit) + lu, 0.f);
    if (!GRAD) return;
    const float cu = (native ? wk * tt : wc) / zs, cw = native ? wk * tt / zt : 0.f;
    each([&](int c, const float(&a)[kChunk], const float(&b)[kChunk]) {
        float y[kChunk];
#pragma unroll
        for (int e = 0; e < kChunk; ++e) {
            y[e] = cu * exp2_((a[e] - ms) * kx);
            if (native) y[e] -= cw * exp2_((b[e] - mt) * kx);
            else if (c * kChunk + e == r.target) y[e] -= wc;
        }
        store_chunk(g, c, y);
    });
}

// one workgroup: sum_i c_main ce_i, c_main kl_i, c_dec kl_i, c_turn kl_i in a fixed order
__global__ __launch_bounds__(kReduceThreads) void distill_reduce_kernel(const DistillRow* rows,
                                                                      const float2* rowval, int n,
                                                                      float* losses) {
    const int tid = threadIdx.x;
    float a = 0.f, b = 0.f, c = 0.f, d = 0.f;
    for (int i = tid; i < n; i += kReduceThreads) {
        const DistillRow r = rows[i];
        const float2 v = rowval[i];
        a += r.target < 0 ? 0.f : r.c_main * v.x;
        b += r.target < 0 ? r.c_main * v.y : 0.f;
        c += r.c_dec * v.y;
        d += r.c_turn * v.y;
    }
    __shared__ float4 sh[kReduceThreads];
    sh[tid] = make_float4(a, b, c, d);
    __syncthreads();
    for (int w = kReduceThreads / 2; w >= 1; w >>= 1) {
        if (tid < w) {
            const float4 x = sh[tid], y = sh[tid + w];
            sh[tid] = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
        }
        __syncthreads();
    }
    if (tid == 0) {
        const float4 t = sh[0];
        losses[0] = t.x;
        losses[1] = t.y;
        losses[2] = t.z;
        losses[3] = t.w;
        losses[4] = ((t.x + t.y) + t.z) + t.w;
    }
}

}  // namespace

// ------------------------------------------------------------------ host API
struct a2t_distill {
    int32_t max_rows = 0, vocab = 0, n_added = 0, dtype = 0, device = 0;
    int cus = 256;
    hipStream_t stream = nullptr;
    DistillRow* rows_dev = nullptr;
    float2* rowval_dev = nullptr;
    DistillRow* stage[2] = {nullptr, nullptr};   // pinned host
    hipEvent_t stage_ev[2] = {nullptr, nullptr};
    bool stage_live[2] = {false, false};
    int next = 0;
    bool poisoned = false;
    // optional dispatch timestamps of the per-row kernel
    bool prof_on = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_pending, prof_free;
    int64_t prof_launches = 0;
    double prof_ms = 0.0;
};

namespace {
struct DevGuard {
    int prev = -1;
    explicit DevGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DevGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};
// Threads of a row's workgroup: as few as hold a row of `chunks` in registers, so that a
// CU has several rows in different phases; more where the rows alone do not fill the
// CUs' 1,024 threads each, as long as a thread keeps four chunks (252 rows of 32,005
// fp32 logits: 20.7 us with 512 threads a row, 24.1 with 1,024, whose waves take
// longer to start; 1,340 rows of 10,009 bf16 logits: 44.8 us with 128, 42.4 with 256),
// and one where they fill less than a quarter (row kernel alone, 27 rows of 3,502 bf16
// logits: 8.3 us with 64 threads, 6.2 with 256; 1,355 of them: 10.3 with 64, 10.7).
int row_threads(int n_rows, int chunks, int regs, int cus) {
    int th = 64;
    const int64_t all = (int64_t)cus * kRowThreads;
    while (th < kRowThreads && th * regs < chunks) th *= 2;
    while (th < kRowThreads && ((8 * th <= chunks && (int64_t)n_rows * th < all) ||
                                (th < 256 && 2 * th <= chunks && 4LL * n_rows * th < all)))
        th *= 2;
    return th;
}
void free_distill(a2t_distill* d) {
    if (!d) return;
    for (int k = 0; k < 2; ++k) {
        if (d->stage_ev[k]) (void)hipEventDestroy(d->stage_ev[k]);
        if (d->stage[k]) (void)hipHostFree(d->stage[k]);
    }
    if (d->rows_dev) (void)hipFree(d->rows_dev);
    if (d->rowval_dev) (void)hipFree(d->rowval_dev);
    for (auto* v : {&d->prof_pending, &d->prof_free})
        for (auto& e : *v) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
    delete d;
}
}  // namespace

extern "C" int a2t_distill_create(int32_t max_rows, int32_t vocab, int32_t n_added, int32_t dtype,
                                  int32_t device, void* hip_stream, a2t_distill** out) {
    if (!out) return A2T_ERR_INVALID;
    *out = nullptr;
    if (max_rows < 1 || vocab < 1 || n_added < 0 || (dtype != A2T_F32 && dtype != A2T_BF16) ||
        (int64_t)vocab + n_added > (1 << 30))
        return A2T_ERR_INVALID;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess || device < 0 || device >= n_dev) return A2T_ERR_NODEV;
    DevGuard g(device);
    a2t_distill* d = new (std::nothrow) a2t_distill();
    if (!d) return A2T_ERR_OOM;
    d->max_rows = max_rows;
    d->vocab = vocab;
    d->n_added = n_added;
    d->dtype = dtype;
    d->device = device;
    d->stream = static_cast<hipStream_t>(hip_stream);
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0) d->cus = cus;
    bool ok = hipMalloc(&d->rows_dev, sizeof(DistillRow) * (size_t)max_rows) == hipSuccess &&
              hipMalloc(&d->rowval_dev, sizeof(float2) * (size_t)max_rows) == hipSuccess;
    for (int k = 0; k < 2 && ok; ++k)
        ok = hipHostMalloc(&d->stage[k], sizeof(DistillRow) * (size_t)max_rows, hipHostMallocDefault) ==
                 hipSuccess &&
             hipEventCreateWithFlags(&d->stage_ev[k], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        free_distill(d);
        return A2T_ERR_OOM;
    }
    *out = d;
    return A2T_OK;
}

extern "C" int a2t_distill_destroy(a2t_distill* d) {
    if (!d) return A2T_ERR_INVALID;
    {
        DevGuard g(d->device);
        (void)hipStreamSynchronize(d->stream);
    }
    free_distill(d);
    return A2T_OK;
}

extern "C" int a2t_distill_loss(a2t_distill* d, int32_t n_rows, const void* student,
                                int64_t student_stride, const void* teacher, int64_t teacher_stride,
                                const int8_t* kind, const int32_t* target, const int8_t* dec_group,
                                const int8_t* turn_group, float temperature, float* losses,
                                void* grad) {
    if (!d) return A2T_ERR_INVALID;
    if (d->poisoned) return A2T_ERR_HIP;
    const int vs = d->vocab + d->n_added;
    if (n_rows < 1 || n_rows > d->max_rows || !student || !teacher || !kind || !target ||
        !dec_group || !turn_group || !losses)
        return A2T_ERR_INVALID;
    if (student_stride < vs || teacher_stride < d->vocab || student_stride % 8 || teacher_stride % 8)
        return A2T_ERR_INVALID;
    auto misaligned = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
    if (misaligned(student) || misaligned(teacher) || (grad && misaligned(grad)) ||
        (reinterpret_cast<uintptr_t>(losses) & 3u))
        return A2T_ERR_INVALID;
    if (!(temperature > 0.f) || !std::isfinite(temperature)) return A2T_ERR_INVALID;
    // row coefficients of the four means (Sec. 3.2)
    int64_t n_asr = 0, n_nat = 0, n_dec[3] = {0, 0, 0}, n_turn[2] = {0, 0};
    for (int i = 0; i < n_rows; ++i) {
        const int k = kind[i];
        if (k < A2T_ROW_NONE || k > A2T_ROW_NATIVE) return A2T_ERR_INVALID;
        if (dec_group[i] < -1 || dec_group[i] > 2 || turn_group[i] < -1 || turn_group[i] > 1)
            return A2T_ERR_INVALID;
        if (k == A2T_ROW_ASR) {
            if (target[i] < 0 || target[i] >= vs) return A2T_ERR_INVALID;
            ++n_asr;
        } else if (k == A2T_ROW_NATIVE) {
            ++n_nat;
            if (dec_group[i] >= 0) ++n_dec[dec_group[i]];
            if (turn_group[i] >= 0) ++n_turn[turn_group[i]];
        }
    }
    const int g_dec = (n_dec[0] > 0) + (n_dec[1] > 0) + (n_dec[2] > 0);
    const int g_turn = (n_turn[0] > 0) + (n_turn[1] > 0);
    DevGuard gd(d->device);
    const int slot = d->next;
    d->next ^= 1;
    if (d->stage_live[slot]) {
        if (hipEventSynchronize(d->stage_ev[slot]) != hipSuccess) {
            d->poisoned = true;
            return A2T_ERR_HIP;
        }
        d->stage_live[slot] = false;
    }
    // rows in order of falling cost (native rows read the teacher too, rows without loss
    // only write zeros), so that the last ones to be dispatched are the short ones
    DistillRow* h = d->stage[slot];
    int at[3] = {(int)(n_nat + n_asr), (int)n_nat, 0};   // by kind: none, ASR, native
    for (int i = 0; i < n_rows; ++i) {
        DistillRow r{i, -1, 0.f, 0.f, 0.f};
        if (kind[i] == A2T_ROW_ASR) {
            r.target = target[i];
            r.c_main = (float)(1.0 / (double)n_asr);
        } else if (kind[i] == A2T_ROW_NATIVE) {
            r.c_main = (float)(1.0 / (double)n_nat);
            if (dec_group[i] >= 0) r.c_dec = (float)(1.0 / ((double)g_dec * n_dec[dec_group[i]]));
            if (turn_group[i] >= 0) r.c_turn = (float)(1.0 / ((double)g_turn * n_turn[turn_group[i]]));
        }
        h[at[kind[i]]++] = r;
    }
    hipError_t e = hipMemcpyAsync(d->rows_dev, h, sizeof(DistillRow) * (size_t)n_rows,
                                  hipMemcpyHostToDevice, d->stream);
    if (e == hipSuccess) e = hipEventRecord(d->stage_ev[slot], d->stream);
    if (e == hipSuccess) d->stage_live[slot] = true;
    const float inv_t = 1.f / temperature;
    if (e == hipSuccess) {
        std::pair<hipEvent_t, hipEvent_t> ev{nullptr, nullptr};
        if (d->prof_on) {
            if (d->prof_free.empty()) {
                hipEvent_t a = nullptr, b = nullptr;
                if (hipEventCreate(&a) == hipSuccess && hipEventCreate(&b) == hipSuccess)
                    d->prof_free.push_back({a, b});
            }
            if (!d->prof_free.empty()) {
                ev = d->prof_free.back();
                d->prof_free.pop_back();
            }
        }
        const int chunks = (vs + kChunk - 1) / kChunk;
        auto go = [&](auto kernel, auto* logits, int th) {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(logits)>>;
            hipExtLaunchKernelGGL(kernel, dim3(n_rows), dim3(th), grad ? th * 128 : 0, d->stream, ev.first, ev.second, 0,
                                  static_cast<const T*>(student), student_stride, static_cast<const T*>(teacher),
                                  teacher_stride, d->vocab, vs, (const DistillRow*)d->rows_dev, inv_t, d->rowval_dev,
                                  static_cast<T*>(grad));
        };
        // the kernel whose threads have few rounds more than the row asks for, because every
        // round is loaded and cut, used or not (row kernel alone, with gradient, 22 rows of 1,715
        // bf16 logits: 10.6 us with 19 rounds, 7.1 with 4; 33 rows of 22,267: 16.5 with 19, 11.8
        // with 8; branches around the rounds made the 19-round kernel spill)
        auto sized = [&](auto* logits) {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(logits)>>;
            constexpr int kRegs = Hold<T>::kRegs, kSome = kRegs > 8 + 4 ? 8 : 4;
            const int th = row_threads(n_rows, chunks, kRegs, d->cus), rounds = (chunks + th - 1) / th;
            auto pick = [&](auto with_grad) {
                constexpr bool G = decltype(with_grad)::value;
                if (rounds <= 4) go(distill_row_kernel<T, G, 4>, logits, th);
                else if (rounds <= kSome) go(distill_row_kernel<T, G, kSome>, logits, th);
                else go(distill_row_kernel<T, G, kRegs>, logits, th);
            };
            if (grad) pick(std::true_type{});
            else pick(std::false_type{});
        };
        if (d->dtype == A2T_F32) sized((const float*)nullptr);
        else sized((const bf16_t*)nullptr);
        e = hipGetLastError();
        if (ev.first) d->prof_pending.push_back(ev);
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(distill_reduce_kernel, dim3(1), dim3(kReduceThreads), 0, d->stream,
                           d->rows_dev, d->rowval_dev, n_rows, losses);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        d->poisoned = true;
        return A2T_ERR_HIP;
    }
    return A2T_OK;
}

extern "C" int a2t_distill_profile_enable(a2t_distill* d, int32_t enable) {
    if (!d) return A2T_ERR_INVALID;
    d->prof_on = enable != 0;
    return A2T_OK;
}

extern "C" int a2t_distill_profile_reserve(a2t_distill* d, int32_t n_launches) {
    if (!d || n_launches < 0) return A2T_ERR_INVALID;
    DevGuard g(d->device);
    while ((int64_t)d->prof_free.size() < (int64_t)n_launches) {
        hipEvent_t a = nullptr, b = nullptr;
        if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
            if (a) (void)hipEventDestroy(a);
            (void)hipGetLastError();
            return A2T_ERR_OOM;
        }
        d->prof_free.push_back({a, b});
    }
    return A2T_OK;
}

extern "C" int a2t_distill_kernel_time(a2t_distill* d, int64_t* launches, double* total_ms) {
    if (!d || !launches || !total_ms) return A2T_ERR_INVALID;
    DevGuard g(d->device);
    for (auto& e : d->prof_pending) {
        if (hipEventSynchronize(e.second) != hipSuccess) return A2T_ERR_HIP;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, e.first, e.second) == hipSuccess) {
            d->prof_launches += 1;
            d->prof_ms += ms;
        }
        d->prof_free.push_back(e);
    }
    d->prof_pending.clear();
    *launches = d->prof_launches;
    *total_ms = d->prof_ms;
    d->prof_launches = 0;
    d->prof_ms = 0.0;
    return A2T_OK;
}
