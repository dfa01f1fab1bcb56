// General path: fp32 storage at any head width D <= 256, and bf16 storage at widths other than 64.  All arithmetic in
// fp32, the products on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: 32 cycles for 2048 operations, twice the
// rate of the vector unit's fused multiply-adds, and one operand register feeds 16 rows).
//
// Bound by the fp32 matrix pipe at sizes that fill the chip, by the length of a wavefront's chain of key blocks below.
// No LDS in the loops: operands go from global memory (L2) to registers, so the wavefronts of a workgroup need no
// barrier, and the four of them SPLIT THE KEYS of the same 16 CQ query rows (blocks w, w + 4, ...): calls on this path
// are short clips in full precision with few rows, which one row range per wavefront would leave most of the chip out
// of.  They merge once, through LDS, at the end; the merge order is fixed, so results are bit-reproducible.
// Measured, 12 heads, 4 frames of 336 tokens, fp32, D = 64 (before: one wavefront per row, operands one element at a
// time): forward 562 -> 44 us, backward 2173 -> 161 us (matrix pipe busy 46-49 % of the cycles); at 32 heads, 8 frames the
// forward reaches 101 TFLOP/s and the backward 103 TFLOP/s of executed products (busy 62-70 %) of the 157 of the instruction.
//
// Lane = (j, g), j = lane % 16, g = lane / 16.  A[i][k] and B[k][j] of the instruction sit in lane i (or j) + 16 k, one
// register each; D[i][j] in lane j + 16 (i / 4), element i % 4.
//   S^T[key, query] = K . Q^T        step (m, e) contracts features 16 m + 4 k + e: one 16-byte load per m and lane
//                                    D: query j, keys 4 g + e of the 16-key block
//   O^T[f, query] += V^T . P^T       step e contracts keys 4 k + e: B = the accumulators as they are; A row i of block
//                                    (c, b) is feature 16 NF c + NF i + b: one load of NF features per lane and e
//                                    D: query j, features 16 NF c + NF (4 g + e) + b
// The gradients use the same two patterns.
//
// A pair that the mask excludes has weight zero, but the second pattern multiplies all 16 rows of a block into all 16
// columns, and zero times an infinity or a NaN is a NaN: what a later frame holds must not reach an earlier one.  A block
// that crosses a bound is therefore looked through first (one fma an element), and if it holds such a value it is
// accumulated once per distinct bound of the workgroup's columns, the rows past that bound set to zero, each column
// keeping the sums of its own pass.
//
// DP: head width rounded up to 32, 64, 128 or 256.  LOAD, how features are loaded (those past D are zero):
//   kWhole   D == DP, tensors 16-byte aligned: vectors of four (two at DP = 32, second pattern)
//   kGroups  D a multiple of four, tensors 16-byte aligned: the same vectors, each of them below D or past it.  One by one
//            they took bf16, D = 96, 12 heads, 4 frames of 336: forward 280 us, backward 980, against 99 and 331
//   kSingle  anything else: one by one
#pragma once
#include "nfd_common.hpp"

namespace nfd {
namespace general {

constexpr int kWaves = 4;
constexpr int kMaxD = 256;

template <typename T> __device__ __forceinline__ T from_f32(float x) { return (T)x; }  // RNE for bf16

enum { kSingle, kGroups, kWhole };
// N consecutive features of a row, as stored where they are loaded as one vector.
template <typename T, int LOAD, int N>
struct Group {
    typedef __attribute__((ext_vector_type(N))) typename std::conditional<LOAD != kSingle, T, float>::type type;
    static __device__ __forceinline__ type load(const T* row, int f, int D) {
        if constexpr (LOAD == kWhole) {
            return *(const type*)(row + f);
        } else if constexpr (LOAD == kGroups) {
            type x = *(const type*)(row + (f < D ? f : 0));
#pragma unroll
            for (int e = 0; e < N; ++e) x[e] = f < D ? x[e] : 0;
            return x;
        } else {
            type x;
#pragma unroll
            for (int e = 0; e < N; ++e) x[e] = f + e < D ? (float)row[f + e] : 0.f;
            return x;
        }
    }
};

// Widened here and not where the value is used.
__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(__bf16 x) {
    float y = (float)x;
    asm volatile("" : "+v"(y));
    return y;
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Where a product does not write the registers it adds to, the compiler takes those as free at once and keeps no distance to
// a vector instruction that writes them (for the bf16 products it does).  Measured: the distance is needed - with the
// softmax of one column block scheduled into the products of the next, whose accumulators had moved, rows of that block
// came out wrong by percents, differently from run to run.  So no vector instruction is scheduled into a group of products
// (loads are), and the last of them is left to read its operands.
extern "C" __device__ void s_nop(short) __asm("llvm.amdgcn.s.nop");  // (inline assembly is not held by the fences)
__device__ __forceinline__ void begin_products() { __builtin_amdgcn_sched_barrier(0x20); }
__device__ __forceinline__ void pin(f32x4& x) { asm volatile("" : "+v"(x)); }
template <typename X, int N>
__device__ __forceinline__ void pin(X (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) pin(x[i]);
}
template <typename... X>
__device__ __forceinline__ void end_products(X&... x) {  // x: all that the group adds to
    (pin(x), ...);
    __builtin_amdgcn_sched_barrier(0x20);
    s_nop(7);
    __builtin_amdgcn_sched_barrier(0x20);
}
template <int N>
__device__ __forceinline__ void zero(f32x4 (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}

template <int DP>
struct Shape {
    static constexpr int M = DP / 16;              // 16-feature groups
    static constexpr int NF = DP >= 64 ? 4 : DP / 16;
    static constexpr int NC = DP / (16 * NF);
};

// 16 rows as an operand of the first pattern: lane (i, g) holds row i, features 16 m + 4 g + e, as loaded and widened.
template <typename T, int DP, int LOAD>
struct RowRaw {
    typename Group<T, LOAD, 4>::type x[Shape<DP>::M];
    __device__ __forceinline__ void load(const T* row, int g, int D) {
#pragma unroll
        for (int m = 0; m < Shape<DP>::M; ++m) x[m] = Group<T, LOAD, 4>::load(row, 16 * m + 4 * g, D);
    }
};
template <typename T, int DP, int LOAD>
struct RowFrag {
    float x[Shape<DP>::M][4];
    __device__ __forceinline__ void operator=(const RowRaw<T, DP, LOAD>& r) {
#pragma unroll
        for (int m = 0; m < Shape<DP>::M; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[m][e] = widen(r.x[m][e]);
    }
    __device__ __forceinline__ void load(const T* row, int g, int D) {
        RowRaw<T, DP, LOAD> r;
        r.load(row, g, D);
        *this = r;
    }
};
// 16 rows as an operand of the second pattern: lane (i, g) holds rows 4 g + e, features 16 NF c + NF i + b (as stored
// where they were loaded as a vector).
template <typename T, int DP, int LOAD>
struct ColFrag {
    typedef Group<T, LOAD, Shape<DP>::NF> group;
    typename group::type x[4][Shape<DP>::NC];
    template <typename RowPtr>
    __device__ __forceinline__ void load(RowPtr row_ptr, int i, int D) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const T* row = row_ptr(e);
#pragma unroll
            for (int c = 0; c < Shape<DP>::NC; ++c) x[e][c] = group::load(row, 16 * Shape<DP>::NF * c + Shape<DP>::NF * i, D);
        }
    }
    // does any lane of the wavefront hold an infinity or a NaN
    __device__ __forceinline__ bool non_finite() const {
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
                for (int b = 0; b < Shape<DP>::NF; ++b) t = __builtin_fmaf((float)x[e][c][b], 0.f, t);
        return __builtin_amdgcn_ballot_w64(t != 0.f) != 0;
    }
    template <typename Seen>
    __device__ __forceinline__ void zero_unless(Seen seen) {  // seen(e): whether the lane's row e counts
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool s = seen(e);
#pragma unroll
            for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
                for (int b = 0; b < Shape<DP>::NF; ++b) x[e][c][b] = s ? x[e][c][b] : 0;
        }
    }
};
template <int DP>
struct Acc {
    f32x4 x[Shape<DP>::NC][Shape<DP>::NF];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
            for (int b = 0; b < Shape<DP>::NF; ++b) x[c][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void scale(float a) {
#pragma unroll
        for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
            for (int b = 0; b < Shape<DP>::NF; ++b) x[c][b] *= a;
    }
    // plus A times P for the lanes that say so; the others keep their sums whatever the products are
    template <typename Frag>
    __device__ __forceinline__ void add_where(const Frag& a, const f32x4& p, bool mine) {
#pragma unroll
        for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
            for (int b = 0; b < Shape<DP>::NF; ++b) {  // one after the other: four registers more, not all of them twice
                f32x4 t = x[c][b];
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = widen(a.x[e][c][b]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e) t = mfma4(y[e], p[e], t);
                end_products(t);
#pragma unroll
                for (int r = 0; r < 4; ++r) x[c][b][r] = mine ? t[r] : x[c][b][r];
            }
    }
    // into column j of a [16][DP] block in LDS
    __device__ __forceinline__ void store(float* col, int g) const {
#pragma unroll
        for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < Shape<DP>::NF; ++b)
                    col[16 * Shape<DP>::NF * c + Shape<DP>::NF * (4 * g + e) + b] = x[c][b][e];
    }
};
// acc += A times P for every column block.  These accumulators live through the loops and stay where they are in all but the
// kernels that say so: fences cost 10 % (forward 45 -> 50 us at 12 heads, 4 frames of 336, fp32), so only those have them.
template <bool FENCED = false, int DP, typename Frag, int N>
__device__ __forceinline__ void accumulate(Acc<DP> (&acc)[N], const Frag& a, f32x4 (&p)[N]) {
    float x[4][Shape<DP>::NC][Shape<DP>::NF];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
            for (int b = 0; b < Shape<DP>::NF; ++b) x[e][c][b] = widen(a.x[e][c][b]);
    if constexpr (FENCED) {
        pin(p);
        begin_products();
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < Shape<DP>::NC; ++c)
#pragma unroll
                for (int b = 0; b < Shape<DP>::NF; ++b) acc[n].x[c][b] = mfma4(x[e][c][b], p[n][e], acc[n].x[c][b]);
    if constexpr (FENCED) {
#pragma unroll
        for (int n = 0; n < N; ++n) pin(acc[n].x);
        end_products();
    }
}
template <typename Frag, int N>
__device__ __forceinline__ void done(Frag& a, f32x4 (&w)[N]) {  // a block already accumulated: nothing is left to add
    a.zero_unless([](int) { return false; });
    zero(w);
}

// The four rows 4 g + e of a block that starts at row r0 of `base`; past the last one (`n` rows) the last again.
template <bool CLAMP, typename T>
__device__ __forceinline__ auto block_rows(const T* base, int r0, int g, int n, int D) {
    const T* first = base + (int64_t)(r0 + 4 * g) * D;
    return [=](int e) { return CLAMP ? base + (int64_t)min(r0 + 4 * g + e, n - 1) * D : first + e * D; };
}

// Sum of the four wavefronts' [16 C][DP] blocks in LDS, times `factor(row)`, to rows row0 .. (below `limit`) of `dst`.
template <typename T, int DP, int C, typename Factor>
__device__ __forceinline__ void write_sum(const float* s, T* dst, int row0, int limit, int D, Factor factor) {
    for (int x = threadIdx.x; x < 16 * C * DP; x += kWaves * 64) {
        const int r = x / DP, f = x % DP;
        if (row0 + r < limit && f < D) {
            float a = s[x];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) a += s[w * 16 * C * DP + x];
            dst[(int64_t)(row0 + r) * D + f] = from_f32<T>(a * factor(r));
        }
    }
}

// C = columns (query rows, or keys in the dk/dv kernel) per workgroup in units of 16.  Two where the registers of two
// wavefronts per SIMD hold them (DP <= 64) and four workgroups per CU remain: an operand register then feeds two matrix
// instructions, but there is half as much to keep the pipe busy between them.  Measured, one block / two (us, fp32, D = 64; the
// workgroups per CU that two leave): backward 148 / 150 (2.0), 345 / 329 (4.4), 314 / 286 (6), 1254 / 1066 (10.5); forward 40 / 47
// (2.0), 91 / 106 (4.4), 83 / 86 (6), 323 / 322 (10.5), 1389 / 1356 (27) - the forward's line is at eight there; at D = 32 it
// is the same as the backward's: 55 / 51 (4.4), 48 / 49 (6), 183 / 172 (10.5).
__host__ __device__ constexpr int padded_width(int D) { return D <= 32 ? 32 : D <= 64 ? 64 : D <= 128 ? 128 : 256; }
__host__ __forceinline__ int cols_per_workgroup(int64_t rows, int64_t BH, int D, int num_cus, bool forward) {
    const int per_cu = forward && padded_width(D) == 64 && D % 4 == 0 ? 8 : 4;
    return padded_width(D) <= 64 && BH * ((rows + 31) / 32) >= per_cu * num_cus ? 2 : 1;
}

template <typename T, int DP, int LOAD, int CQ>
__global__ void __launch_bounds__(kWaves * 64, DP == 256 ? 1 : DP == 128 && sizeof(T) == 2 && LOAD == kWhole ? 3 : 2)
attn_fwd_general(FwdParams p) {
    __shared__ float o_s[kWaves * 16 * CQ * DP];
    __shared__ float m_s[kWaves][16 * CQ], l_s[kWaves][16 * CQ], inv_s[16 * CQ];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int bh = (int)(blockIdx.x % (unsigned)p.BH);
    const int r0 = (p.n_q_tiles - 1 - (int)(blockIdx.x / (unsigned)p.BH)) * 16 * CQ;  // latest (heaviest) rows first
    const int D = p.D;
    const T* qg = (const T*)p.q + (int64_t)bh * p.Sq * D;
    const T* kg = (const T*)p.k + (int64_t)bh * p.Scap * D;
    const T* vg = (const T*)p.v + (int64_t)bh * p.Scap * D;
    RowFrag<T, DP, LOAD> qf[CQ];
    Acc<DP> o[CQ];
    float m[CQ], l[CQ];
    int kmax_lane[CQ];
#pragma unroll
    for (int c = 0; c < CQ; ++c) {
        const int rc = min(r0 + 16 * c + j, p.Sq - 1);  // ragged tail: a duplicate row, never stored
        qf[c].load(qg + (int64_t)rc * D, g, D);
        o[c].zero();
        m[c] = kNegBig;
        l[c] = 0.f;
        kmax_lane[c] = kmax_of_row(rc, p.T, p.P);
    }
    const int kmin = kmax_of_row(min(r0, p.Sq - 1), p.T, p.P), kmax = kmax_of_row(min(r0 + 16 * CQ, p.Sq) - 1, p.T, p.P);
    const int n_blk = (kmax + 15) / 16;
    // The next block's keys are requested before this block's products where that costs no resident wavefront (wide
    // heads: 726 against 778 us at 32 heads, 8 frames of 336, D = 128), behind them otherwise (D = 64: 314 against 318).
    constexpr bool PREFETCH = DP > 64;
    RowRaw<T, DP, LOAD> kr;  // the next block's keys, widened when their turn comes
    if (wave < n_blk) kr.load(kg + (int64_t)min(16 * wave + j, p.Sk - 1) * D, g, D);
    auto block = [&](int b, auto masked) {
        const int j0 = 16 * b;
        ColFrag<T, DP, LOAD> vf;
        vf.load(block_rows<masked>(vg, j0, g, p.Sk, D), j, D);
        RowFrag<T, DP, LOAD> kf;
        kf = kr;
        if (PREFETCH && b + kWaves < n_blk) kr.load(kg + (int64_t)min(j0 + 16 * kWaves + j, p.Sk - 1) * D, g, D);
        f32x4 s[CQ];
        zero(s);
        begin_products();
#pragma unroll
        for (int m = 0; m < Shape<DP>::M; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < CQ; ++c) s[c] = mfma4(kf.x[m][e], qf[c].x[m][e], s[c]);
        end_products(s);
#pragma unroll
        for (int c = 0; c < CQ; ++c) {
            if (masked) {
                const int left = kmax_lane[c] - (j0 + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e >= left) s[c][e] = -INFINITY;
            }
            s[c] *= p.scale_log2e;
            float a = fmaxf(fmaxf(s[c][0], s[c][1]), fmaxf(s[c][2], s[c][3]));
            a = fmaxf(a, __shfl_xor(a, 16));
            a = fmaxf(a, __shfl_xor(a, 32));
            const float m_new = fmaxf(m[c], a);
            const float alpha = exp2f(m[c] - m_new);
            m[c] = m_new;
#pragma unroll
            for (int e = 0; e < 4; ++e) s[c][e] = exp2f(s[c][e] - m_new);
            l[c] = l[c] * alpha + ((s[c][0] + s[c][1]) + (s[c][2] + s[c][3]));
            if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) o[c].scale(alpha);
        }
        if (masked && vf.non_finite()) {
            for (int bound = kmax; bound >= kmin && bound > j0; bound -= p.T) {  // latest frame first: ever fewer rows count
                vf.zero_unless([&](int e) { return j0 + 4 * g + e < bound; });
#pragma unroll
                for (int c = 0; c < CQ; ++c) o[c].add_where(vf, s[c], kmax_lane[c] == bound);
            }
            done(vf, s);
        }
        accumulate(o, vf, s);
        if (!PREFETCH && b + kWaves < n_blk) kr.load(kg + (int64_t)min(j0 + 16 * kWaves + j, p.Sk - 1) * D, g, D);
    };
    int b = wave;
    for (; b < n_blk && 16 * b + 16 <= kmin; b += kWaves) block(b, std::false_type{});
    for (; b < n_blk; b += kWaves) block(b, std::true_type{});
#pragma unroll
    for (int c = 0; c < CQ; ++c) {
        l[c] += __shfl_xor(l[c], 16);
        l[c] += __shfl_xor(l[c], 32);
        if (g == 0) {
            m_s[wave][16 * c + j] = m[c];
            l_s[wave][16 * c + j] = l[c];
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CQ; ++c) {
        float mm = m_s[0][16 * c + j];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, m_s[w][16 * c + j]);
        o[c].scale(exp2f(m[c] - mm));
        o[c].store(o_s + (wave * 16 * CQ + 16 * c + j) * DP, g);
    }
    if ((int)threadIdx.x < 16 * CQ) {  // one thread per row: the merged row sum
        const int r = threadIdx.x;
        float mm = m_s[0][r], ll = 0.f;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, m_s[w][r]);
#pragma unroll
        for (int w = 0; w < kWaves; ++w) ll += l_s[w][r] * exp2f(m_s[w][r] - mm);
        inv_s[r] = 1.0f / ll;
        if (p.lse && r0 + r < p.Sq) p.lse[(int64_t)bh * p.Sq + r0 + r] = (mm + log2f(ll)) * kLn2;
    }
    __syncthreads();
    write_sum<T, DP, CQ>(o_s, (T*)p.out + (int64_t)bh * p.Sq * D, r0, p.Sq, D, [&](int r) { return inv_s[r]; });
}

// Backward.  With p_ij = exp(scale <q_i, k_j> - lse_i) over the visible keys of row i and delta_i = <dout_i, out_i>:
// ds_ij = p_ij (<dout_i, v_j> - delta_i), dq_i = scale sum_j ds_ij k_j, dk_j = scale sum_i ds_ij q_i,
// dv_j = sum_i p_ij dout_i.  Two kernels, neither with atomics; the dq kernel first (it writes delta).
struct BwdParams {
    const void *q, *k, *v, *out, *dout;
    const float* lse;
    float* delta;  // [BH, Sq], written by the dq kernel, read by the dk/dv kernel
    void *dq, *dk, *dv;
    int BH, Sq, Sk, Scap, T, P, D;
    int n_q_tiles, n_k_tiles;
    float scale, scale_log2e;
};

template <typename T, int DP, int LOAD, int CQ>
__global__ void __launch_bounds__(kWaves * 64, DP == 256 ? 1 : 2)
attn_bwd_dq_general(BwdParams p) {
    __shared__ float o_s[kWaves * 16 * CQ * DP];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int bh = (int)(blockIdx.x % (unsigned)p.BH);
    const int r0 = (p.n_q_tiles - 1 - (int)(blockIdx.x / (unsigned)p.BH)) * 16 * CQ;
    const int D = p.D;
    const T* kg = (const T*)p.k + (int64_t)bh * p.Scap * D;
    const T* vg = (const T*)p.v + (int64_t)bh * p.Scap * D;
    RowFrag<T, DP, LOAD> qf[CQ], gf[CQ];
    Acc<DP> dq[CQ];
    float lse2[CQ], delta[CQ];
    int kmax_lane[CQ];
#pragma unroll
    for (int c = 0; c < CQ; ++c) {
        const int row = r0 + 16 * c + j, rc = min(row, p.Sq - 1);
        const int64_t at = ((int64_t)bh * p.Sq + rc) * D;
        qf[c].load((const T*)p.q + at, g, D);
        gf[c].load((const T*)p.dout + at, g, D);
        RowFrag<T, DP, LOAD> of;
        of.load((const T*)p.out + at, g, D);
        float a = 0.f;
#pragma unroll
        for (int m = 0; m < Shape<DP>::M; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) a = fmaf(gf[c].x[m][e], of.x[m][e], a);
        a += __shfl_xor(a, 16);
        delta[c] = a + __shfl_xor(a, 32);
        if (wave == 0 && g == 0 && row < p.Sq) p.delta[(int64_t)bh * p.Sq + row] = delta[c];
        lse2[c] = p.lse[(int64_t)bh * p.Sq + rc] * kLog2e;
        dq[c].zero();
        kmax_lane[c] = kmax_of_row(rc, p.T, p.P);
    }
    const int kmin = kmax_of_row(min(r0, p.Sq - 1), p.T, p.P), kmax = kmax_of_row(min(r0 + 16 * CQ, p.Sq) - 1, p.T, p.P);
    const int n_blk = (kmax + 15) / 16;
    auto block = [&](int b, auto masked) {
        const int j0 = 16 * b;
        RowFrag<T, DP, LOAD> kf, vf;
        const int64_t at = (int64_t)(masked ? min(j0 + j, p.Sk - 1) : j0 + j) * D;
        kf.load(kg + at, g, D);
        vf.load(vg + at, g, D);
        ColFrag<T, DP, LOAD> kt;
        kt.load(block_rows<masked>(kg, j0, g, p.Sk, D), j, D);
        f32x4 s[CQ], dp[CQ];
        zero(s);
        zero(dp);
        begin_products();
#pragma unroll
        for (int m = 0; m < Shape<DP>::M; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < CQ; ++c) {
                    s[c] = mfma4(kf.x[m][e], qf[c].x[m][e], s[c]);
                    dp[c] = mfma4(vf.x[m][e], gf[c].x[m][e], dp[c]);
                }
        end_products(s, dp);
#pragma unroll
        for (int c = 0; c < CQ; ++c) {
            const int left = masked ? kmax_lane[c] - (j0 + 4 * g) : 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float pr = exp2f(s[c][e] * p.scale_log2e - lse2[c]);
                dp[c][e] = e < left ? pr * (dp[c][e] - delta[c]) : 0.f;
            }
        }
        if (masked && kt.non_finite()) {
            for (int bound = kmax; bound >= kmin && bound > j0; bound -= p.T) {  // latest frame first: ever fewer rows count
                kt.zero_unless([&](int e) { return j0 + 4 * g + e < bound; });
#pragma unroll
                for (int c = 0; c < CQ; ++c) dq[c].add_where(kt, dp[c], kmax_lane[c] == bound);
            }
            done(kt, dp);
        }
        accumulate(dq, kt, dp);
    };
    int b = wave;
    for (; b < n_blk && 16 * b + 16 <= kmin; b += kWaves) block(b, std::false_type{});
    for (; b < n_blk; b += kWaves) block(b, std::true_type{});
#pragma unroll
    for (int c = 0; c < CQ; ++c) dq[c].store(o_s + (wave * 16 * CQ + 16 * c + j) * DP, g);
    __syncthreads();
    write_sum<T, DP, CQ>(o_s, (T*)p.dq + (int64_t)bh * p.Sq * D, r0, p.Sq, D, [&](int) { return p.scale; });
}

// dk, dv: a workgroup owns 16 CK keys, its wavefronts split the 16-row blocks of queries that see them.  A lane holds
// key column j and rows 4 g + e of a block.  Key j is visible to row i iff i >= (floor(j/T) - P) T: the blocks that cross a
// bound are the first ones (passes from the earliest frame on), and a ragged last one.
template <typename T, int DP, int LOAD, int CK>
__global__ void __launch_bounds__(kWaves * 64, DP == 256 ? 1 : 2)
attn_bwd_dkdv_general(BwdParams p) {
    __shared__ float o_s[kWaves * 16 * CK * DP];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int bh = (int)(blockIdx.x % (unsigned)p.BH);
    const int k0 = (int)(blockIdx.x / (unsigned)p.BH) * 16 * CK;  // earliest keys (seen by most rows) first
    const int D = p.D;
    const T* qg = (const T*)p.q + (int64_t)bh * p.Sq * D;
    const T* gg = (const T*)p.dout + (int64_t)bh * p.Sq * D;
    const float* lse = p.lse + (int64_t)bh * p.Sq;
    const float* delta = p.delta + (int64_t)bh * p.Sq;
    RowFrag<T, DP, LOAD> kf[CK], vf[CK];
    Acc<DP> dk[CK], dv[CK];
    int rmin_lane[CK];
    auto first_row = [&](int key) { return max(0, (key / p.T - p.P) * p.T); };  // the first row that sees the key
#pragma unroll
    for (int c = 0; c < CK; ++c) {
        const int kc = min(k0 + 16 * c + j, p.Sk - 1);
        const int64_t at = ((int64_t)bh * p.Scap + kc) * D;
        kf[c].load((const T*)p.k + at, g, D);
        vf[c].load((const T*)p.v + at, g, D);
        dk[c].zero();
        dv[c].zero();
        rmin_lane[c] = first_row(kc);
    }
    constexpr bool FENCED = CK == 2 && (DP == 32 || sizeof(T) == 2);  // here the compiler moves dv and dk (see accumulate)
    constexpr bool EARLY = DP <= 64;  // all four operands of a block are requested at once where the registers hold them
    const int rmin = first_row(k0), rmax = first_row(min(k0 + 16 * CK, p.Sk) - 1);
    const int b0 = rmin / 16, b1 = (p.Sq + 15) / 16;
    auto block = [&](int b, auto masked) {
        const int i0 = 16 * b;
        f32x4 s[CK], dp[CK];
        ColFrag<T, DP, LOAD> tg, tq;
        float lse2[4], dl[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int ic = masked ? min(i0 + 4 * g + e, p.Sq - 1) : i0 + 4 * g + e;
            lse2[e] = lse[ic];
            dl[e] = delta[ic];
        }
        {
            RowFrag<T, DP, LOAD> qa, ga;
            const int64_t at = (int64_t)(masked ? min(i0 + j, p.Sq - 1) : i0 + j) * D;
            qa.load(qg + at, g, D);
            ga.load(gg + at, g, D);
            if (EARLY) {
                tg.load(block_rows<masked>(gg, i0, g, p.Sq, D), j, D);
                tq.load(block_rows<masked>(qg, i0, g, p.Sq, D), j, D);
            }
            zero(s);
            zero(dp);
            begin_products();
#pragma unroll
            for (int m = 0; m < Shape<DP>::M; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int c = 0; c < CK; ++c) {
                        s[c] = mfma4(qa.x[m][e], kf[c].x[m][e], s[c]);
                        dp[c] = mfma4(ga.x[m][e], vf[c].x[m][e], dp[c]);
                    }
            end_products(s, dp);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + 4 * g + e;
#pragma unroll
            for (int c = 0; c < CK; ++c) {
                const bool seen = !masked || (i >= rmin_lane[c] && i < p.Sq);
                const float pr = seen ? exp2f(s[c][e] * p.scale_log2e - lse2[e] * kLog2e) : 0.f;
                s[c][e] = pr;
                dp[c][e] = seen ? pr * (dp[c][e] - dl[e]) : 0.f;
            }
        }
        auto add = [&](ColFrag<T, DP, LOAD>& t, Acc<DP>(&acc)[CK], f32x4(&w)[CK]) {
            if (masked && t.non_finite()) {
                t.zero_unless([&](int e) { return i0 + 4 * g + e < p.Sq; });
                for (int bound = rmin; bound <= rmax && bound < i0 + 16; bound += p.T) {
                    t.zero_unless([&](int e) { return i0 + 4 * g + e >= bound; });
#pragma unroll
                    for (int c = 0; c < CK; ++c) acc[c].add_where(t, w[c], rmin_lane[c] == bound);
                }
                done(t, w);
            }
            accumulate<FENCED>(acc, t, w);
        };
        if (!EARLY) tg.load(block_rows<masked>(gg, i0, g, p.Sq, D), j, D);
        add(tg, dv, s);
        if (!EARLY) tq.load(block_rows<masked>(qg, i0, g, p.Sq, D), j, D);
        add(tq, dk, dp);
    };
    int b = b0 + wave;
    for (; b < b1 && 16 * b < rmax; b += kWaves) block(b, std::true_type{});
    for (; b < b1 && 16 * b + 16 <= p.Sq; b += kWaves) block(b, std::false_type{});
    for (; b < b1; b += kWaves) block(b, std::true_type{});
#pragma unroll
    for (int c = 0; c < CK; ++c) dk[c].store(o_s + (wave * 16 * CK + 16 * c + j) * DP, g);
    __syncthreads();
    write_sum<T, DP, CK>(o_s, (T*)p.dk + (int64_t)bh * p.Scap * D, k0, p.Sk, D, [&](int) { return p.scale; });
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CK; ++c) dv[c].store(o_s + (wave * 16 * CK + 16 * c + j) * DP, g);
    __syncthreads();
    write_sum<T, DP, CK>(o_s, (T*)p.dv + (int64_t)bh * p.Scap * D, k0, p.Sk, D, [](int) { return 1.0f; });
}

}  // namespace general
}  // namespace nfd
