// MFMA fragments in fragment order and the GEMM epilogues, shared by the streaming
// (gemm_decode.hip) and the LDS-tiled (gemm_tiled.hip) kernels.
#pragma once

#include "common.h"
#include "kernels.h"

namespace aed {

template <typename T> struct Frag16;
template <> struct Frag16<bf16_t> { bf16x8 lo, hi; };
template <> struct Frag16<float> { float v[16]; };

// a lane's 16 k-values of one block in fragment order: pieces at stride 1 KB
__device__ __forceinline__ Frag16<bf16_t> load_frag(const bf16_t* blk, int lane) {
    Frag16<bf16_t> f;
    const bf16x8* p = reinterpret_cast<const bf16x8*>(blk) + lane;
    f.lo = p[0];
    f.hi = p[64];
    return f;
}
__device__ __forceinline__ Frag16<bf16_t> load_frag_nt(const bf16_t* blk, int lane) {
    Frag16<bf16_t> f;
    const bf16x8* p = reinterpret_cast<const bf16x8*>(blk) + lane;
    f.lo = __builtin_nontemporal_load(p);
    f.hi = __builtin_nontemporal_load(p + 64);
    return f;
}
__device__ __forceinline__ Frag16<float> load_frag(const float* blk, int lane) {
    Frag16<float> f;
    const f32x4* p = reinterpret_cast<const f32x4*>(blk) + lane;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f32x4 v = p[64 * j];
        f.v[4 * j + 0] = v[0]; f.v[4 * j + 1] = v[1]; f.v[4 * j + 2] = v[2]; f.v[4 * j + 3] = v[3];
    }
    return f;
}
__device__ __forceinline__ Frag16<float> load_frag_nt(const float* blk, int lane) { return load_frag(blk, lane); }
// A 16-row tile of a fragment-order operand, n_rows rows of it present.  Lanes of absent rows point past the descriptor's
// end: such a load returns zeros and asks memory for nothing.  K up to kMaxK; beyond, 16 rows have more bytes than the
// descriptor's offsets reach, and a product takes tiles of more rows (choose_tile).
template <int ES> struct FragRows {
    static constexpr int kEnd = 0x40000000;  // offsets of present rows are below (16 rows of K elements), of absent ones above
    static constexpr int kMaxK = kEnd / (16 * ES);
    __amdgpu_buffer_rsrc_t rsrc;
    int voff;  // this lane's bytes within a 1 KB piece
    __device__ __forceinline__ FragRows(const char* base, int n_rows, int lane)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, kEnd, 0x20000)),
          voff((lane & 15) < n_rows ? lane * 16 : 0x7ffffff0) {}
    __device__ __forceinline__ void load(int kb, Frag16<bf16_t>& f) const {
        f.lo = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, kb * 2048, 0));
        f.hi = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, kb * 2048 + 1024, 0));
    }
    __device__ __forceinline__ void load(int kb, Frag16<float>& f) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, kb * 4096 + 1024 * j, 0));
            f.v[4 * j + 0] = v[0]; f.v[4 * j + 1] = v[1]; f.v[4 * j + 2] = v[2]; f.v[4 * j + 3] = v[3];
        }
    }
};
__device__ __forceinline__ void pack_frag(const float* y, Frag16<bf16_t>& f) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { f.lo[i] = (bf16_t)y[i]; f.hi[i] = (bf16_t)y[8 + i]; }
}
__device__ __forceinline__ void unpack_frag(const Frag16<bf16_t>& f, float* y) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { y[i] = (float)f.lo[i]; y[8 + i] = (float)f.hi[i]; }
}
// acc[n-major 16x16] += W-fragment x A-fragment over the 64-wide k block
__device__ __forceinline__ void mma(f32x4& acc, const Frag16<bf16_t>& w, const Frag16<bf16_t>& a) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.lo, a.lo, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.hi, a.hi, acc, 0, 0, 0);
}
// Four consecutive cache elements as 8-bit E4M3 codes (OCP 8-bit floating point: bias 7, no infinities, largest
// magnitude 448): round to nearest even, done by the conversion instruction; saturation is done here.
__device__ __forceinline__ void store4_fp8(unsigned char* p, f32x4 s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = fminf(fmaxf(s[i], -448.f), 448.f);
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(s[0], s[1], 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(s[2], s[3], w, true);
    *reinterpret_cast<int*>(p) = w;
}

// (mean, sum of squared deviations) of a row from four tiles per lane of the 16 lanes that share it; every lane gets it.
// EXACT: the sum of the tiles' means, each as large as the row's common offset, has roundings of that size; what the means are away
// from its result is exact, and its mean is what the result lacks.  (4 layers in float32, rows 10 spreads from zero: error of the
// logits 9.9e-7 without, 9.3e-7 with it, a step 0.5 to 1 % longer.)
template <bool EXACT = false> __device__ __forceinline__ float2 combine_tile_stats(f32x4 u, f32x4 v, bool live, int tiles) {
    float mu = row16_sum(live ? (u[0] + u[2]) + (v[0] + v[2]) : 0.f) / (float)tiles;
    float d0 = u[0] - mu, d1 = u[2] - mu, d2 = v[0] - mu, d3 = v[2] - mu;
    if constexpr (EXACT) {
        const float rest = row16_sum(live ? (d0 + d1) + (d2 + d3) : 0.f) / (float)tiles;
        mu += rest;
        d0 -= rest; d1 -= rest; d2 -= rest; d3 -= rest;
    }
    const float q = (u[1] + u[3]) + (v[1] + v[3]) + 16.f * ((d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3));
    return float2{mu, row16_sum(live ? q : 0.f)};
}
// Mean and sum of squared deviations of rows [m0, m0 + BM) over all columns, from the 16-column tiles' (GemmArgs::stats_in),
// into LDS; 256 threads, 16 lanes per row.  Mean of the tiles' means, then the tiles' own sums of squares plus
// 16 x the squared distances of their means.  All loads first: one round trip.
template <int BM> __device__ __forceinline__ void load_row_stats(const GemmArgs& a, int m0, float2* row_stat) {
    constexpr int P = BM / 16;
    const int row = threadIdx.x >> 4, t4 = 4 * (threadIdx.x & 15);
    const bool live = t4 < a.stat_tiles;
    f32x4 v[P][2];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const f32x4* sp = reinterpret_cast<const f32x4*>(a.stats_in + (size_t)(m0 + 16 * p + row) * a.stat_tiles +
                                                         min(t4, a.stat_tiles - 4));
        v[p][0] = sp[0];
        v[p][1] = sp[1];
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const float2 st = combine_tile_stats(v[p][0], v[p][1], live, a.stat_tiles);
        if ((threadIdx.x & 15) == 0) row_stat[16 * p + row] = st;
    }
}

// Where row m goes in the caches (rows from M on: anywhere valid, they are not stored)
template <int EPI> __device__ __forceinline__ int row_slot(const GemmArgs& a, int m) {
    if constexpr (EPI == EPI_QKV) return a.kv_slot[min(m, a.M - 1)];
    else if constexpr (EPI == EPI_CROSSKV) return a.out_row_map ? a.out_row_map[min(m, a.M - 1)] : m;
    else return -1;
}

// One lane's four consecutive outputs C[m][n .. n+3] (bias already added) go where the epilogue says.
// slot: EPI_QKV: kv_slot[m], EPI_CROSSKV: the frame
// of row m -- read by the caller once per row, ahead of the stores.
template <typename T, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int m, int n, f32x4 s, int slot) {
    constexpr int ES = sizeof(T);
    if constexpr (EPI == EPI_F32) {
        store4(static_cast<float*>(a.out) + (size_t)m * a.N + n, s);
    } else if constexpr (EPI == EPI_RELU_T) {
        s[0] = fmaxf(s[0], 0.f); s[1] = fmaxf(s[1], 0.f); s[2] = fmaxf(s[2], 0.f); s[3] = fmaxf(s[3], 0.f);
        store4(reinterpret_cast<T*>(static_cast<char*>(a.out) + frag_elem_off<ES>(m, n, a.N)), s);
    } else if constexpr (EPI == EPI_QKV) {
        const int d = a.d_model;
        if (n < d) {
            store4(static_cast<float*>(a.out) + (size_t)m * d + n, s);
        } else if (slot >= 0) {
            const int which = n >= 2 * d;
            const int c = n - (which ? 2 * d : d), sh = a.head_dim == 128 ? 7 : 6;
            const int h = c >> sh, e = c & (a.head_dim - 1);
            const size_t at = ((((size_t)(slot >> 4) * a.n_heads + h) * kPage + (slot & 15)) << sh) + e;
            if (a.kv_fp8) store4_fp8(static_cast<unsigned char*>(which ? a.v_pool : a.k_pool) + at, s);
            else store4(static_cast<T*>(which ? a.v_pool : a.k_pool) + at, s);
        }
    } else {  // EPI_CROSSKV
        const int d = a.d_model;
        const int which = n >= d;
        const int c = n - (which ? d : 0), sh = a.head_dim == 128 ? 7 : 6;
        const int h = c >> sh, e = c & (a.head_dim - 1);
        const size_t at = (((size_t)h * a.t_cap + slot) << sh) + e;
        if (a.kv_fp8) store4_fp8(static_cast<unsigned char*>(which ? a.vc : a.kc) + at, s);
        else store4(static_cast<T*>(which ? a.vc : a.kc) + at, s);
    }
}

}  // namespace aed
