// Cross-attention over the encoder frames themselves (bfloat16, d_model 1024, 8 heads of 128), for large batches.
//
// With keys K = E Wk^T + bk and values V = E Wv^T + bv of the frames E, a head's scores and output are
//   q . K_t        = (Wk^T q) . E_t + q . bk       (the last term is the same for every frame: the softmax drops it)
//   sum_t p_t V_t  = Wv (sum_t p_t E_t) + bv       (the p_t add up to 1)
// so a step can read the frames, 2 KB each and the same for all heads, where it reads 4 KB of keys and values per frame.  At
// large batches that stream is what bounds cross-attention; the price are two small products per row and layer
// (frames_query_kernel, frames_out_kernel) and 8 times the multiplications of one query row, which go to the matrix cores.
//
// The matrix cores take bfloat16.  The frames are bfloat16; what is float32 goes in as two of them, high and low
// (x = hi + lo up to 2^-17): the 8 heads' queries Wk^T q fill the 16 columns of a 16 x 16 tile as 8 high and 8 low parts, the
// probabilities likewise, and the frames' weighted sums enter the last product as high and low parts.  Sums are float32.
// The rounding of keys and values to bfloat16 is gone.
#include <algorithm>

#include "common.h"
#include "gemm_common.h"
#include "kernels.h"
#include "device_once.h"

namespace aed {

namespace {

constexpr int kD = 1024, kH = 8, kDh = 128, kCols = 16;
constexpr int kSlab = 16384, kPart = 8192;               // bytes of LDS: a wavefront's part of 32 frames; all wavefronts' partial scores of a position
constexpr int kNonTemporal = 2;  // a buffer load's nt bit: the frames are read once and should not push other data out of the caches
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split(float x, bf16_t& hi, bf16_t& lo) {
    hi = (bf16_t)x;
    lo = (bf16_t)(x - (float)hi);
}
__device__ __forceinline__ float other_half(float v) { return dpp_mov<0x128>(v); }  // of lane l ^ 8 (row_ror 8)

}  // namespace

// ---------------------------------------------------------------- Wk^T q
// Q[b][c][k], 16 x 1024 a row: for head h the high (c = h) and low (c = 8 + h) parts of scale * sum_e q[b][128 h + e] Wk[128 h + e][k].
// A workgroup takes 32 rows, 256 of the 1024 columns k and one head; the products are short (K = 128), so what counts is the
// 32 KB a row that are written: row i = 4 g + e of a wavefront's weight tile t is column 16 g + 4 t + e of its 64, so that a lane
// ends with 16 consecutive columns and four lanes write whole lines.  Heads are dealt to the XCDs (x = 8 heads).
// Wt: per head [1024][128] in fragment order (launch_frames_weight).
__global__ __launch_bounds__(256) void frames_query_kernel(const float* __restrict__ q, const char* __restrict__ Wt, bf16_t* __restrict__ Q,
                                                           int M, float scale) {
    constexpr int MT = 2, NT = 4;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int h = blockIdx.x, n0 = blockIdx.y * 256 + wave * 64, m0 = blockIdx.z * 32;
    Frag16<bf16_t> w[NT][2];
    const char* wp = Wt + (size_t)h * kD * kDh * 2 + frag_block_off<2>((n0 >> 4) + (r >> 2), 0, kDh);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) w[nt][kb] = load_frag(reinterpret_cast<const bf16_t*>(wp + kb * 2048), g * 16 + 4 * nt + (r & 3));
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        // lane (r, g) takes elements 16 j + 4 g .. + 3 of a 64-wide block, so that four lanes read 64 bytes in a row; Wt is stored to match
        const f32x4* p = reinterpret_cast<const f32x4*>(q + (size_t)min(m0 + mt * 16 + r, M - 1) * kD + h * kDh + g * 4);
        float x[2][16];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 v = p[kb * 16 + j * 4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[kb][4 * j + e] = v[e];
            }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            Frag16<bf16_t> hi, lo;
            float res[16];
            pack_frag(x[kb], hi);
            unpack_frag(hi, res);
#pragma unroll
            for (int e = 0; e < 16; ++e) res[e] = x[kb][e] - res[e];
            pack_frag(res, lo);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                mma(acc[mt][nt], w[nt][kb], hi);
                mma(acc[mt][nt], w[nt][kb], lo);
            }
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + mt * 16 + r;
        if (m >= M) continue;
        bf16_t* out = Q + ((size_t)m * kCols + h) * kD + n0 + 16 * g;
        bf16x8 hi[2], lo[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            bf16_t a, b;
            split(acc[mt][e >> 2][e & 3] * scale, a, b);
            hi[e >> 3][e & 7] = a;
            lo[e >> 3][e & 7] = b;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            *reinterpret_cast<bf16x8*>(out + 8 * j) = hi[j];
            *reinterpret_cast<bf16x8*>(out + kH * kD + 8 * j) = lo[j];
        }
    }
}

// ---------------------------------------------------------------- attention
// One workgroup per sequence, all heads.  U[b][c][k]: high and low parts of head h's sum_t p_t E[t][k], as Q.
// Bound by memory: a sequence's frames are read once, 2 KB each.  A step takes 32 frames; wavefront w has columns 256 w .. + 255
// of them:
//  * frames come from fragment order (the encoder states as the cross K/V product reads them, so a sequence's first and last
//    16-row tile may hold its neighbours' frames, which are masked) straight into registers: rows of a tile = frames, the
//    operand of the score product, Q's part staying in registers (32 of them);
//  * the four wavefronts' partial scores are added through LDS (the step's only barrier; two buffers), every wavefront then
//    has all 32 frames' scores and takes the softmax itself: lane (c, g) holds frames 4 g .. 4 g + 3 of either tile for column c,
//    which is the operand layout of the second product;
//  * the second product contracts over frames, so it needs them transposed: each wavefront puts its part into LDS and reads it
//    back through the transposing read (ds_read_b64_tr_b16: 16 lanes read four rows of four 8-byte pieces, lane i gets column i).
//    Piece p of a tile's row is the 4 columns 16 p + 4 t of a 64-column block, so that a lane's sums are 16 consecutive columns
//    after t = 0 .. 3; the quarters of a block are stored 4 rows apart from each other, so that the four pieces lie in different banks;
//  * the next step's frames are requested as soon as this step's are in LDS: 64 KB a workgroup, 128 KB a CU under way.
// A prompt pass has several positions of a sequence: NQ of them are taken at once, with one reading of the frames.
// Q and U begin with row row0.
template <int NQ>
__global__ __launch_bounds__(256, NQ == 1 ? 2 : 1) void attn_frames_kernel(const void* E, const void* Q, const int4* items, void* U, int first, int stride,
                                                                           int row0) {
    extern __shared__ __align__(16) char lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int4 it = items[blockIdx.x * stride + first];
    int b[NQ];
    b[0] = it.x;
#pragma unroll
    for (int i = 1; i < NQ; ++i) b[i] = items[blockIdx.x * stride + first + i].x;
    if (b[0] < 0) return;  // the sequence has finished (kItemOff)
#pragma unroll
    for (int i = 0; i < NQ; ++i) b[i] -= row0;
    const int n = it.z & 0xFFFF, skip = it.w & 15;
    const int tiles = (skip + n + 15) >> 4, steps = (tiles + 1) >> 1;
    const char* src = static_cast<const char*>(E) + (size_t)(it.w >> 4) * (kD * 32) + wave * 8192;
    char* slab = lds + wave * kSlab;
    char* part = lds + 4 * kSlab;

    bf16x8 x[2][8];  // a step's two tiles, 8 pieces of 16 bytes a lane each
    // through a buffer descriptor: of a tile past the end, requested all the same so that no request sits behind a branch, the
    // lanes ask beyond the descriptor's end and nothing is fetched (65535 frames are 128 MB)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, 0x40000000, 0x20000);
    auto fetch = [&](int s, int u) {
        const int t = 2 * s + u, at = t < tiles ? t * (kD * 32) : 0, voff = t < tiles ? lane * 16 : 0x7ffffff0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            x[u][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, at + j * 1024, kNonTemporal));
        __builtin_amdgcn_sched_barrier(0);
    };
    bf16x8 qf[NQ][8];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const bf16_t* p = static_cast<const bf16_t*>(Q) + ((size_t)b[i] * kCols + r) * kD + wave * 256 + 16 * g;
#pragma unroll
        for (int j = 0; j < 8; ++j) qf[i][j] = *reinterpret_cast<const bf16x8*>(p + (j >> 1) * 64 + (j & 1) * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch(0, 0);
    fetch(0, 1);
    f32x4 acc[NQ][4][4];  // [.][m][t], lane (c, g): columns 64 m + 16 g + 4 t .. + 3 of this wavefront's 256, for column c of Q
#pragma unroll
    for (int i = 0; i < NQ; ++i)
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[i][m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run[NQ], l_run[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) { m_run[i] = -INFINITY; l_run[i] = 0.f; }
    char* const put = slab + g * 256 + (r ^ (4 * g)) * 16;
    const auto get = (__attribute__((address_space(3))) char*)slab + (r & 3) * 256 + ((4 * g + (r >> 2)) ^ (4 * (r & 3))) * 16;

#pragma unroll 1
    for (int s = 0; s < steps; ++s) {
        char* const buf = part + (s & 1) * (NQ * kPart);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            // scores of this wavefront's columns
            f32x4 sc[NQ];
#pragma unroll
            for (int i = 0; i < NQ; ++i) sc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int i = 0; i < NQ; ++i) sc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][j], qf[i][j], sc[i], 0, 0, 0);
            // the frames into LDS, zeros in the place of those that are not this sequence's (their probability is 0, but 0
            // times an infinity is not); then the next step's are requested
            const int t = (2 * s + u) * 16 + r - skip;
            const bool own = t >= 0 && t < n;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                u32x4 v = __builtin_bit_cast(u32x4, x[u][j]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = own ? v[e] : 0u;
                *reinterpret_cast<u32x4*>(put + u * 8192 + j * 1024) = v;
            }
            fetch(s + 1, u);
#pragma unroll
            for (int i = 0; i < NQ; ++i) *reinterpret_cast<f32x4*>(buf + i * kPart + wave * 2048 + u * 1024 + lane * 16) = sc[i];
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
        bf16x8 pf[NQ];
        float alpha[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            // all columns' scores; high and low part of the query together
            float p[2][4], m_blk = -INFINITY;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x4 v[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const f32x4*>(buf + i * kPart + w * 2048 + u * 1024 + lane * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float d = (v[0][e] + v[1][e]) + (v[2][e] + v[3][e]);
                    d += other_half(d);
                    const int t = (2 * s + u) * 16 + 4 * g + e - skip;
                    p[u][e] = t >= 0 && t < n ? d : -INFINITY;
                    m_blk = fmaxf(m_blk, p[u][e]);
                }
            }
            m_blk = rows4_max(m_blk);
            const float m_new = fmaxf(m_run[i], m_blk);
            alpha[i] = __builtin_amdgcn_exp2f(m_run[i] - m_new);  // first step: exp2(-inf) = 0
            m_run[i] = m_new;
            l_run[i] *= alpha[i];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = __builtin_amdgcn_exp2f(p[u][e] - m_new);
                    l_run[i] += v;
                    bf16_t hi, lo;
                    split(v, hi, lo);
                    pf[i][4 * u + e] = r < kH ? hi : lo;
                }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                // frames 4 g .. 4 g + 3 of both tiles, column 64 m + 16 (r / 4) + 4 t + r % 4
                u32x2 a[2];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    a[u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) s16x4*)(get + u * 8192 + m * 2048 + (t >> 1) * 1024 + (t & 1) * 8)));
                const bf16x8 e8 = __builtin_bit_cast(bf16x8, u32x4{a[0][0], a[0][1], a[1][0], a[1][1]});
#pragma unroll
                for (int i = 0; i < NQ; ++i) acc[i][m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e8, pf[i], acc[i][m][t] * alpha[i], 0, 0, 0);
            }
        other_lanes_wrote();  // the next step's frames go where these were read from (in front of the reads stands the barrier)
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const float inv = 1.0f / rows4_sum(l_run[i]);
        bf16_t* out = static_cast<bf16_t*>(U) + ((size_t)b[i] * kCols + r) * kD + wave * 256 + 16 * g;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float a = acc[i][m][2 * j + (e >> 2)][e & 3], v = (a + other_half(a)) * inv;
                    bf16_t hi, lo;
                    split(v, hi, lo);
                    o[e] = r < kH ? hi : lo;
                }
                *reinterpret_cast<bf16x8*>(out + m * 64 + j * 8) = o;
            }
    }
}

template <int NQ> static hipError_t launch_positions(const FramesArgs& a, int first, int row0, hipStream_t s) {
    constexpr int kLds = 4 * kSlab + 2 * NQ * kPart;
    static DeviceOnce once;
    const hipError_t e = once.run([] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_frames_kernel<NQ>), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_frames_kernel<NQ>, dim3(a.n_items / a.positions), dim3(256), kLds, s, a.frames, a.q_frames, a.items, a.u_frames, first,
                       a.positions, row0);
    return hipGetLastError();
}

// ---------------------------------------------------------------- Wv u + bv
// out[b][128 h + e] (fragment order) = sum_k Wv[128 h + e][k] (U[b][h][k] + U[b][8 + h][k]) + bv.  A workgroup takes 32 rows and half a
// head's 128 columns; the wavefronts split k and their sums meet in LDS, as in gemm_decode.hip.  U is read as it lies: 16 rows of
// 64 contiguous bytes an instruction.
__global__ __launch_bounds__(256, 2) void frames_out_kernel(const bf16_t* __restrict__ U, const char* __restrict__ Wv, const bf16_t* __restrict__ bias,
                                                            char* __restrict__ out, int M) {
    constexpr int MT = 2, NT = 4;
    __shared__ f32x4 sum[4][MT * NT][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int h = blockIdx.x, n0 = blockIdx.y * 64, m0 = blockIdx.z * 32;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a 64-wide block's piece p is k = 32 p + 8 g .. + 7 here, which in the weights' fragment order is quarter 2 p + g / 2, half g % 2
    bf16x8 af[2][MT][2][2], wf[2][NT][2];
    auto fetch = [&](int slot, int i) {
        const int kb = wave * 4 + i;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                wf[slot][nt][p] = *reinterpret_cast<const bf16x8*>(Wv + frag_block_off<2>(((h * kDh + n0) >> 4) + nt, kb, kD) + (g & 1) * 1024 +
                                                                   ((2 * p + (g >> 1)) * 16 + r) * 16);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int part = 0; part < 2; ++part)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    af[slot][mt][part][p] = *reinterpret_cast<const bf16x8*>(
                        U + ((size_t)min(m0 + mt * 16 + r, M - 1) * kCols + part * kH + h) * kD + kb * 64 + p * 32 + g * 8);
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, 0);
    fetch(1, 1);
    f32x4 bv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) bv[i] = bias ? load4(bias + h * kDh + n0 + ((wave + 4 * i) % NT) * 16 + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int part = 0; part < 2; ++part)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i & 1][nt][p], af[i & 1][mt][part][p], acc[mt][nt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (i + 2 < 4) fetch(i & 1, i + 2);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sum[wave][mt * NT + nt][lane] = acc[mt][nt];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = wave + 4 * i, m = m0 + (t / NT) * 16 + r;
        const f32x4 v = (sum[0][t][lane] + sum[1][t][lane]) + (sum[2][t][lane] + sum[3][t][lane]) + bv[i];
        if (m < M) store4(reinterpret_cast<bf16_t*>(out + frag_elem_off<2>(m, h * kDh + n0 + (t % NT) * 16 + 4 * g, kD)), v);
    }
}

// ---------------------------------------------------------------- Wk^T, once at create
// dst: per head [1024][128] in fragment order, element 16 j + 4 g + e of a 64-wide block in the place of 16 g + 4 j + e (see
// frames_query_kernel) <- W [1024 (h, e)][1024 k] row-major; one thread per 16-byte piece
__global__ __launch_bounds__(256) void frames_weight_kernel(const bf16_t* __restrict__ W, char* __restrict__ dst) {
    const int i = blockIdx.x * 256 + threadIdx.x, k = i & (kD - 1), p0 = (i >> 10) * 8;  // neighbours read neighbouring k
    if (p0 >= kD) return;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int p = p0 + e;
        v[e] = W[(size_t)((p & ~63) + 16 * ((p & 15) >> 2) + 4 * ((p & 63) >> 4) + (p & 3)) * kD + k];
    }
    const int h = p0 / kDh;
    *reinterpret_cast<bf16x8*>(dst + (size_t)h * kD * kDh * 2 + frag_elem_off<2>(k, p0 % kDh, kDh)) = v;
}

hipError_t launch_frames_weight(const void* W, void* dst, hipStream_t s) {
    hipLaunchKernelGGL(frames_weight_kernel, dim3(kD * kD / 8 / 256), dim3(256), 0, s, static_cast<const bf16_t*>(W), static_cast<char*>(dst));
    return hipGetLastError();
}

hipError_t launch_attn_frames(const FramesArgs& a, hipStream_t s) {
    if (a.rows < 1 || a.n_items < 1 || !a.items || a.positions < 1 || a.n_items % a.positions != 0 || a.rows % a.positions != 0) return hipErrorInvalidValue;
    const int Bs = a.rows / a.positions;
    if (a.positions > 1 && Bs % 16 != 0) return hipErrorInvalidValue;  // a part of the output begins with a 16-row tile
    // A prompt pass in parts of kFramesPart positions, each with its queries and sums in the same scratch (64 KB a row): a batch has as
    // much of it as four of its steps need, whatever the pass takes.  (1024 sequences in three positions, the two products of a layer:
    // 80 us in one part, 83 in two.)
    for (int part = 0; part < a.positions; part += kFramesPart) {
        const int end = std::min(part + kFramesPart, a.positions), row0 = part * Bs, rows = (end - part) * Bs;
        const unsigned tiles = (rows + 31) / 32;
        hipLaunchKernelGGL(frames_query_kernel, dim3(kH, kD / 256, tiles), dim3(256), 0, s, a.q + (size_t)row0 * kD, static_cast<const char*>(a.wk_t),
                           static_cast<bf16_t*>(a.q_frames), rows, a.scale_log2e);
        hipError_t e = hipGetLastError();
        for (int at = part; at < end && e == hipSuccess; at += 2)  // two with one reading of the frames: of three the sums do not fit the registers
            e = at + 2 <= end ? launch_positions<2>(a, at, row0, s) : launch_positions<1>(a, at, row0, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(frames_out_kernel, dim3(kH, kDh / 64, tiles), dim3(256), 0, s, static_cast<const bf16_t*>(a.u_frames), static_cast<const char*>(a.wv),
                           static_cast<const bf16_t*>(a.bv), static_cast<char*>(a.out) + frag_block_off<2>(row0 / 16, 0, kD), rows);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace aed
