// Streaming kernels: cache copies, window moves and the rotary pre-op.
#pragma once
#include "kernels_fp8.hpp"
#include "nfd_common.hpp"

namespace nfd {

// Copy a run of whole frames of every head between two head-strided tensors: the cache write of new
// frames (Appendix B, KV caching) and the moves of the sliding context window.  K and V together.
// All counts in units of the element type E (a 16-byte vector when every size and address allows it,
// otherwise one tensor element): head_dst / head_src = head strides, off_dst / off_src = offsets
// inside a head, len = units per head.  blockIdx.y walks over the heads, blockIdx.x over the units of a
// head, so no thread divides.
// PAIR = false: one tensor only (kd, ks); vd and vs are not touched.
template <typename E, bool PAIR = true>
__global__ void __launch_bounds__(256)
kvcache_copy(E* __restrict__ kd, E* __restrict__ vd, const E* __restrict__ ks, const E* __restrict__ vs,
             int64_t head_dst, int64_t head_src, int64_t off_dst, int64_t off_src, int64_t len, int64_t heads) {
    for (int64_t bh = blockIdx.y; bh < heads; bh += gridDim.y) {
        const int64_t dbase = bh * head_dst + off_dst, sbase = bh * head_src + off_src;
        for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < len; r += (int64_t)gridDim.x * blockDim.x) {
            kd[dbase + r] = ks[sbase + r];
            if constexpr (PAIR) vd[dbase + r] = vs[sbase + r];
        }
    }
}

// Slide a window inside its tensor in one pass: units [d, d + len) of every row move to [0, len), d = units dropped.
// Bound by memory: every kept byte is read once and written once (a copy out to the workspace and back, which this
// replaces where it is faster, moves everything twice).  Few kept units that land where only dropped ones were are copied
// instead (kvcache_copy; rule and figures at shift_copied on the host).  Two ways to keep a unit from being overwritten
// before it is read:
//  * chains, for rows with many units to drop (heads of K, V): units r, r + d, r + 2d, ... form a chain, each
//    overwritten by the next one of the same chain and by nothing else, so one thread walks one chain front to back,
//    U units at a time (all U read before the first is written), with no order between threads;
//  * whole rows, for the short feature rows of the 8-bit V cache (a chain would touch 16 bytes per row): a workgroup
//    owns a row and moves it front to back in pieces of 256 x U units, a barrier between reading and writing a piece.
// PERM: units are single keys of the 8-bit V cache (frames that are no multiple of its 16-key groups), whose positions
// go through the permuted order inside a group.
// Measured, 16 heads, 32 frames of 336 tokens kept, two dropped: K and V in bf16 (44 MB read, 44 MB written, part of it in
// the last-level cache) 13.5 us against 27.9 through the workspace; the 8-bit caches 7.4 against 26.5.
struct ShiftRun {
    void* base;
    int64_t stride;  // units per row (a head, or a feature row of the 8-bit V cache)
    int64_t rows, d, len;
};
template <typename E>
__device__ __forceinline__ void shift_chains(const ShiftRun& a, int64_t block) {
    constexpr int U = 8;
    const int64_t idx = block * 256 + threadIdx.x;
    if (idx >= a.rows * a.d) return;
    const int64_t row = idx <= 0xffffffffll && a.d <= 0xffffffffll ? (int64_t)((uint32_t)idx / (uint32_t)a.d) : idx / a.d;
    E* base = (E*)a.base + row * a.stride;
    int64_t x = idx - row * a.d;
    for (; x + (U - 1) * a.d < a.len; x += U * a.d) {
        E r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = base[x + (u + 1) * a.d];
#pragma unroll
        for (int u = 0; u < U; ++u) base[x + u * a.d] = r[u];
    }
    E r[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (x + u * a.d < a.len) r[u] = base[x + (u + 1) * a.d];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (x + u * a.d < a.len) base[x + u * a.d] = r[u];
}
template <typename E, bool PERM>
__device__ __forceinline__ void shift_row(const ShiftRun& a, int64_t row) {
    constexpr int U = 8;
    const int s = (int)((row >> 4) & 1);  // rows are (head, feature): bit 4 of the feature
    E* base = (E*)a.base + row * a.stride;
    auto at = [&](int64_t x) -> E& { return base[PERM ? v8t_position(x, s) : x]; };
    for (int64_t x0 = 0; x0 < a.len; x0 += 256 * U) {
        E r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t x = x0 + 256 * u + threadIdx.x;
            if (x < a.len) r[u] = at(x + a.d);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t x = x0 + 256 * u + threadIdx.x;
            if (x < a.len) at(x) = r[u];
        }
        __syncthreads();
    }
}
// Heads of two tensors of one geometry, as chains (blocks below nblk0: the first tensor).  `first`: the launch's first block, as
// very large windows take several.
template <typename E>
__global__ void __launch_bounds__(256)
kvcache_shift_inplace(ShiftRun a, ShiftRun b, int64_t nblk0, int64_t first) {
    const int64_t block = first + blockIdx.x;
    if (block < nblk0) shift_chains<E>(a, block);
    else shift_chains<E>(b, block - nblk0);
}
// The 8-bit caches: heads of K codes as chains, feature rows of V codes whole.
template <typename EK, typename EV, bool PERM>
__global__ void __launch_bounds__(256)
kvcache_shift_fp8_inplace(ShiftRun k, ShiftRun v, int64_t nblk0, int64_t first) {
    const int64_t block = first + blockIdx.x;
    if (block < nblk0) shift_chains<EK>(k, block);
    else shift_row<EV, PERM>(v, block - nblk0);
}

// ---------------------------------------------------------------------------------------------
// 3D rotary position embedding of the queries and keys of the new frames, fused with the cache
// write (Sec. 3.1 "3D Positional Embedding": the head dimension is separated into [n_T, n_H, n_W],
// one rotary embedding per axis, concatenated; Appendix B for the cache).  The rotation of feature
// pair (2i, 2i+1) of an axis section of width n at position p is by the angle p * theta^(-2i/n),
// counter-clockwise.  Pure streaming work: q in -> q out, k -> cache, v -> cache.
//
// One thread owns VEC consecutive features of one (frame, token) and walks over a range of heads:
// the cosines and sines depend on the position only, so they are computed once (in fp64: angles
// reach hundreds of radians) and reused for every head.  Consecutive threads cover consecutive
// 16-byte chunks of consecutive tokens, i.e. contiguous memory inside each head.
constexpr int kRopeMaxPairs = 128;  // D <= 256
struct RopeTable {
    double inv_freq[kRopeMaxPairs];     // theta^(-2i/n) of every feature pair, in head-dimension order
    unsigned char axis[kRopeMaxPairs];  // 0 = frame index, 1 = grid row, 2 = grid column
};
struct RopeParams {
    int BH, F, T, D;
    int frame_pos, n_frames;
    int t_pos0;            // temporal position of the first new frame
    int grid_w;
    int heads_per_thread;  // blockIdx.y selects a range of heads
};

//
// KV8 (bf16, VEC = 8 only): the caches are the 8-bit ones (kernels_fp8.hpp): the rotated key, rounded to bf16
// exactly as for a bf16 cache, and the value are quantised with the head's scales; K codes go to 8 consecutive
// bytes of the key's row, V codes to 8 feature rows at the key's (permuted) position.
struct RopeFp8 {
    const float* k_scale;  // [BH]
    const float* v_scale;  // [BH]
    int64_t Spad;          // keys per cache row set (F * T rounded up to 64)
};

template <typename E, int VEC, bool KV8 = false>
__global__ void __launch_bounds__(256)
rope_kvcache_append(const E* q, E* q_out, E* __restrict__ kc, E* __restrict__ vc,
                    const E* __restrict__ kn, const E* __restrict__ vn, RopeParams rp, RopeTable tab, RopeFp8 f8 = RopeFp8{}) {
    typedef __attribute__((ext_vector_type(VEC))) E vec_t;
    const int chunks = rp.D / VEC;
    const int64_t items = (int64_t)rp.n_frames * rp.T * chunks;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= items) return;
    const int chunk = (int)(idx % chunks);
    const int64_t row = idx / chunks;  // (new frame, token)
    const int f = (int)(row / rp.T), tok = (int)(row % rp.T);
    const int pos[3] = {rp.t_pos0 + f, tok / rp.grid_w, tok % rp.grid_w};
    float cs[VEC / 2], sn[VEC / 2];
#pragma unroll
    for (int j = 0; j < VEC / 2; ++j) {
        const int p = chunk * (VEC / 2) + j;
        const double ang = (double)pos[tab.axis[p]] * tab.inv_freq[p];
        double s, c;
        sincos(ang, &s, &c);
        cs[j] = (float)c;
        sn[j] = (float)s;
    }
    const int bh0 = blockIdx.y * rp.heads_per_thread;
    const int bh1 = min(bh0 + rp.heads_per_thread, rp.BH);
    for (int bh = bh0; bh < bh1; ++bh) {
        const int64_t src = ((int64_t)bh * rp.n_frames * rp.T + row) * rp.D + chunk * VEC;
        const int64_t dst = (((int64_t)bh * rp.F + rp.frame_pos) * rp.T + row) * rp.D + chunk * VEC;
        const vec_t qv = *(const vec_t*)(q + src);
        const vec_t kv = *(const vec_t*)(kn + src);
        const vec_t vv = *(const vec_t*)(vn + src);
        vec_t qo, ko;
#pragma unroll
        for (int j = 0; j < VEC / 2; ++j) {
            const float qa = (float)qv[2 * j], qb = (float)qv[2 * j + 1];
            const float ka = (float)kv[2 * j], kb = (float)kv[2 * j + 1];
            qo[2 * j] = (E)(qa * cs[j] - qb * sn[j]);
            qo[2 * j + 1] = (E)(qa * sn[j] + qb * cs[j]);
            ko[2 * j] = (E)(ka * cs[j] - kb * sn[j]);
            ko[2 * j + 1] = (E)(ka * sn[j] + kb * cs[j]);
        }
        *(vec_t*)(q_out + src) = qo;
        if constexpr (KV8) {
            static_assert(!KV8 || VEC == 8, "the 8-bit cache takes eight features per thread");
            const float ik = __frcp_rn(f8.k_scale[bh]), iv = __frcp_rn(f8.v_scale[bh]);
            const int64_t j = (int64_t)rp.frame_pos * rp.T + row;  // key index in the cache
            uint32_t w0 = e4m3_pack2<false>((float)ko[0] * ik, (float)ko[1] * ik, 0u);
            w0 = e4m3_pack2<true>((float)ko[2] * ik, (float)ko[3] * ik, w0);
            uint32_t w1 = e4m3_pack2<false>((float)ko[4] * ik, (float)ko[5] * ik, 0u);
            w1 = e4m3_pack2<true>((float)ko[6] * ik, (float)ko[7] * ik, w1);
            const u32x2 w = {w0, w1};
            *(u32x2*)((unsigned char*)kc + ((int64_t)bh * f8.Spad + j) * 64 + chunk * 8) = w;
            unsigned char* vd = (unsigned char*)vc + ((int64_t)bh * 64 + chunk * 8) * f8.Spad + v8t_position(j, (chunk >> 1) & 1);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                vd[(int64_t)e * f8.Spad] = (unsigned char)(e4m3_pack2<false>((float)vv[e] * iv, 0.f, 0u) & 0xffu);
        } else {
            *(vec_t*)(kc + dst) = ko;
            *(vec_t*)(vc + dst) = vv;
        }
    }
}

}  // namespace nfd
