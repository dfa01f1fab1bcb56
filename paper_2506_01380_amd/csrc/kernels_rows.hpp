// General path, few rows or keys a head: one wavefront owns one query row (one key row in the dk/dv kernel) and walks what it
// sees 64 at a time, a lane per key for the scores and a lane per feature for the sums, fp32 arithmetic on the vector
// unit.  Bound by latency and by a serial loop over the features; but a row is all a workgroup's quarter computes, where
// the tile kernels fill 16 x 16 blocks, widths of 32 to 256 and four wavefronts however few of each are there (the rule
// and its figures are at GeneralPrice on the host).
#pragma once
#include "kernels_general.hpp"

namespace nfd {
namespace rows {

template <typename T> __device__ __forceinline__ float to_f32(T x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<__bf16>(__bf16 x) { return (float)x; }
using general::from_f32;

__device__ __forceinline__ float wave_max(float x) {
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

constexpr int kRowsPerWorkgroup = 4;

template <typename T>
__global__ void __launch_bounds__(kRowsPerWorkgroup * 64)
attn_fwd_rows(FwdParams p) {
    __shared__ float q_s[kRowsPerWorkgroup][general::kMaxD];
    __shared__ float p_s[kRowsPerWorkgroup][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t row_id = (int64_t)blockIdx.x * kRowsPerWorkgroup + w;  // over BH * Sq
    if (row_id >= (int64_t)p.BH * p.Sq) return;                          // whole wave exits together
    const int bh = (int)(row_id / p.Sq), i = (int)(row_id % p.Sq);
    const int D = p.D;
    const T* q = (const T*)p.q + ((int64_t)bh * p.Sq + i) * D;
    const T* k = (const T*)p.k + (int64_t)bh * p.Scap * D;
    const T* v = (const T*)p.v + (int64_t)bh * p.Scap * D;
    T* out = (T*)p.out + ((int64_t)bh * p.Sq + i) * D;

    for (int d = lane; d < D; d += 64) q_s[w][d] = to_f32<T>(q[d]);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): q_s visible within the wave

    const int kmax = kmax_of_row(i, p.T, p.P);  // <= Sk by construction
    float m = kNegBig, l = 0.f;
    float acc[general::kMaxD / 64] = {0.f, 0.f, 0.f, 0.f};

    for (int j0 = 0; j0 < kmax; j0 += 64) {
        const int j = j0 + lane;
        float s = -INFINITY;
        if (j < kmax) {
            const T* kr = k + (int64_t)j * D;
            float a = 0.f;
            for (int d = 0; d < D; ++d) a = fmaf(q_s[w][d], to_f32<T>(kr[d]), a);
            s = a * p.scale_log2e;  // log2 units
        }
        const float m_new = fmaxf(m, wave_max(s));
        const float alpha = exp2f(m - m_new);
        const float pj = exp2f(s - m_new);  // 0 for masked lanes
        l = l * alpha + wave_sum(pj);
        m = m_new;
        p_s[w][lane] = pj;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(0xc07f);
        const int nj = min(64, kmax - j0);
#pragma unroll
        for (int c = 0; c < general::kMaxD / 64; ++c) {
            const int d = lane + 64 * c;
            if (d < D) {
                float a = acc[c] * alpha;
                for (int jj = 0; jj < nj; ++jj) a = fmaf(p_s[w][jj], to_f32<T>(v[(int64_t)(j0 + jj) * D + d]), a);
                acc[c] = a;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int c = 0; c < general::kMaxD / 64; ++c) {
        const int d = lane + 64 * c;
        if (d < D) out[d] = from_f32<T>(acc[c] * inv);
    }
    if (p.lse && lane == 0) p.lse[row_id] = (m + log2f(l)) * kLn2;
}

// Backward (definitions at the tile kernels' in kernels_general.hpp): two kernels, neither with atomics, the dq kernel first (it
// writes delta).
// One wavefront per query row: delta_i, then dq_i over the visible keys, 64 at a time.
template <typename T>
__global__ void __launch_bounds__(kRowsPerWorkgroup * 64)
attn_bwd_dq_rows(general::BwdParams p) {
    __shared__ float q_s[kRowsPerWorkgroup][general::kMaxD];
    __shared__ float g_s[kRowsPerWorkgroup][general::kMaxD];
    __shared__ float ds_s[kRowsPerWorkgroup][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t row_id = (int64_t)blockIdx.x * kRowsPerWorkgroup + w;  // over BH * Sq
    if (row_id >= (int64_t)p.BH * p.Sq) return;
    const int bh = (int)(row_id / p.Sq), i = (int)(row_id % p.Sq);
    const int D = p.D;
    const T* q = (const T*)p.q + row_id * D;
    const T* o = (const T*)p.out + row_id * D;
    const T* g = (const T*)p.dout + row_id * D;
    const T* k = (const T*)p.k + (int64_t)bh * p.Scap * D;
    const T* v = (const T*)p.v + (int64_t)bh * p.Scap * D;

    float dsum = 0.f;
    for (int d = lane; d < D; d += 64) {
        const float gd = to_f32<T>(g[d]);
        q_s[w][d] = to_f32<T>(q[d]);
        g_s[w][d] = gd;
        dsum = fmaf(gd, to_f32<T>(o[d]), dsum);
    }
    const float delta = wave_sum(dsum);
    if (lane == 0) p.delta[row_id] = delta;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);

    const float lse2 = p.lse[row_id] * kLog2e;
    const int kmax = kmax_of_row(i, p.T, p.P);
    float acc[general::kMaxD / 64] = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < kmax; j0 += 64) {
        const int j = j0 + lane;
        float ds = 0.f;
        if (j < kmax) {
            const T* kr = k + (int64_t)j * D;
            const T* vr = v + (int64_t)j * D;
            float a = 0.f, b = 0.f;
            for (int d = 0; d < D; ++d) {
                a = fmaf(q_s[w][d], to_f32<T>(kr[d]), a);
                b = fmaf(g_s[w][d], to_f32<T>(vr[d]), b);
            }
            ds = exp2f(a * p.scale_log2e - lse2) * (b - delta);
        }
        ds_s[w][lane] = ds;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(0xc07f);
        const int nj = min(64, kmax - j0);
#pragma unroll
        for (int c = 0; c < general::kMaxD / 64; ++c) {
            const int d = lane + 64 * c;
            if (d < D) {
                float a = acc[c];
                for (int jj = 0; jj < nj; ++jj) a = fmaf(ds_s[w][jj], to_f32<T>(k[(int64_t)(j0 + jj) * D + d]), a);
                acc[c] = a;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    T* dq = (T*)p.dq + row_id * D;
#pragma unroll
    for (int c = 0; c < general::kMaxD / 64; ++c) {
        const int d = lane + 64 * c;
        if (d < D) dq[d] = from_f32<T>(acc[c] * p.scale);
    }
}

// One wavefront per key row j < Sk: dk_j and dv_j over the query rows that see it, 64 at a time.  Those are
// the rows from (floor(j/T) - P) * T on (none below 0): every later frame sees the key as well.
template <typename T>
__global__ void __launch_bounds__(kRowsPerWorkgroup * 64)
attn_bwd_dkdv_rows(general::BwdParams p) {
    __shared__ float k_s[kRowsPerWorkgroup][general::kMaxD];
    __shared__ float v_s[kRowsPerWorkgroup][general::kMaxD];
    __shared__ float p_s[kRowsPerWorkgroup][64];
    __shared__ float ds_s[kRowsPerWorkgroup][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t key_id = (int64_t)blockIdx.x * kRowsPerWorkgroup + w;  // over BH * Sk
    if (key_id >= (int64_t)p.BH * p.Sk) return;
    const int bh = (int)(key_id / p.Sk), j = (int)(key_id % p.Sk);
    const int D = p.D;
    const T* kr = (const T*)p.k + ((int64_t)bh * p.Scap + j) * D;
    const T* vr = (const T*)p.v + ((int64_t)bh * p.Scap + j) * D;
    const T* q = (const T*)p.q + (int64_t)bh * p.Sq * D;
    const T* g = (const T*)p.dout + (int64_t)bh * p.Sq * D;
    const float* lse = p.lse + (int64_t)bh * p.Sq;
    const float* delta = p.delta + (int64_t)bh * p.Sq;

    for (int d = lane; d < D; d += 64) {
        k_s[w][d] = to_f32<T>(kr[d]);
        v_s[w][d] = to_f32<T>(vr[d]);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);

    const int rmin = max(0, (j / p.T - p.P) * p.T);
    float acc_k[general::kMaxD / 64] = {0.f, 0.f, 0.f, 0.f};
    float acc_v[general::kMaxD / 64] = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = rmin; i0 < p.Sq; i0 += 64) {
        const int i = i0 + lane;
        float pij = 0.f, ds = 0.f;
        if (i < p.Sq) {
            const T* qr = q + (int64_t)i * D;
            const T* gr = g + (int64_t)i * D;
            float a = 0.f, b = 0.f;
            for (int d = 0; d < D; ++d) {
                a = fmaf(to_f32<T>(qr[d]), k_s[w][d], a);
                b = fmaf(to_f32<T>(gr[d]), v_s[w][d], b);
            }
            pij = exp2f(a * p.scale_log2e - lse[i] * kLog2e);
            ds = pij * (b - delta[i]);
        }
        p_s[w][lane] = pij;
        ds_s[w][lane] = ds;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(0xc07f);
        const int ni = min(64, p.Sq - i0);
#pragma unroll
        for (int c = 0; c < general::kMaxD / 64; ++c) {
            const int d = lane + 64 * c;
            if (d < D) {
                float ak = acc_k[c], av = acc_v[c];
                for (int ii = 0; ii < ni; ++ii) {
                    ak = fmaf(ds_s[w][ii], to_f32<T>(q[(int64_t)(i0 + ii) * D + d]), ak);
                    av = fmaf(p_s[w][ii], to_f32<T>(g[(int64_t)(i0 + ii) * D + d]), av);
                }
                acc_k[c] = ak;
                acc_v[c] = av;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    T* dk = (T*)p.dk + ((int64_t)bh * p.Scap + j) * D;
    T* dv = (T*)p.dv + ((int64_t)bh * p.Scap + j) * D;
#pragma unroll
    for (int c = 0; c < general::kMaxD / 64; ++c) {
        const int d = lane + 64 * c;
        if (d < D) {
            dk[d] = from_f32<T>(acc_k[c] * p.scale);
            dv[d] = from_f32<T>(acc_v[c]);
        }
    }
}

}  // namespace rows
}  // namespace nfd
