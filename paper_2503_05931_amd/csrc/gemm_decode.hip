// Weight-streaming MFMA GEMM for the decoder step's projections (QKV, attention
// output, cross-attention query, FFN, vocabulary) on gfx950.
//
// C[M,N] = prologue(A)[M,K] . W[N,K]^T: M is the decode batch (1..1024), the
// weights W are read exactly once per launch and dominate the traffic, so the
// kernel is organised around streaming W:
//   * a workgroup (4 wavefronts; 8 where launch_nb says so) owns a (16*MT) x (16*NT) output tile;
//   * the NW wavefronts split K: wavefront w takes the 64-wide k blocks
//     w, w+NW, w+2 NW, ..., and the partial tiles are summed through LDS in a
//     fixed order (deterministic);
//   * lane (r, g) (r = lane % 16, g = lane / 16) holds, for row r of a 16-row
//     operand, the 16 consecutive k values k0 + 16 g .. +15 of a 64-wide block.
//     Both operands use the same k assignment, so the MFMA's internal k order
//     does not matter;
//   * both operands live in memory in fragment order (common.h): the weights
//     are re-ordered once when the decoder is created, the activations are
//     written in that order by the kernels that produce them.  Every operand
//     load is then one coalesced 1 KB instruction per wavefront straight into
//     MFMA registers -- no LDS staging, no transposes;
//   * the weight fragment is the first MFMA operand: lane (r, g) then holds
//     C[m = r][n = 4 g .. 4 g + 3], four consecutive outputs of one row, which
//     is one 16-byte (fp32) or 8-byte (bf16) store, also into fragment order.
// A LayerNorm before a product is taken around it (kernels.h) in both storage types.  In float32 it was a prologue that
// normalised and kept the rows before the first multiplication (up to 128 rows), or a launch of its own; us a step of 4 layers of
// d_model 1024 with it / with the mean taken off the operands as they arrive: batch 16 233.5 / 187.8, 32 246.6 / 203.5, 128
// 428.9 / 356.9, 256 588.1 / 564.5, 900 1719 / 1726.
#include <algorithm>

#include "common.h"
#include "device_once.h"
#include "gemm_common.h"
#include "kernel_tail.h"
#include "kernels.h"

namespace aed {

// What a workgroup needs before its first request to memory: leading scalar arguments; the rest comes in a tail (kernel_tail.h)
struct GemmStart { const void *W, *A; const float2* stats_in; int M, K, stat_tiles; };
template <typename T, int PRO, int EPI> struct GemmFields {
    static constexpr bool LNS = PRO == PRO_LNS, RS = EPI == EPI_RESID_S, QKV = EPI == EPI_QKV, CKV = EPI == EPI_CROSSKV,
                          ADD = EPI == EPI_F32 && PRO == PRO_T, SHADOW = sizeof(T) == 2;
    template <typename F> __host__ __device__ __forceinline__ static constexpr void fields(GemmArgs& a, F&& f) {
        f(a.out);
        if constexpr (LNS) f(a.ln_c2); else f(a.bias);
        if constexpr (LNS && SHADOW) { f(a.ln_c1); f(a.mu_hat_out); }
        if constexpr (LNS && QKV && SHADOW) { f(a.out2); f(a.raw_bias); }
        if constexpr ((LNS || RS) && SHADOW) f(a.mu_hat_in);
        if constexpr (RS) f(a.stats_out);
        if constexpr (RS && SHADOW) f(a.shadow_out);
        if constexpr (ADD) f(a.addend);
        if constexpr (QKV) { f(a.kv_slot); f(a.k_pool); f(a.v_pool); }
        if constexpr (CKV) { f(a.out_row_map); f(a.kc); f(a.vc); f(a.t_cap); }
        f(a.N);
        if constexpr (LNS) { f(a.rms); f(a.ln_eps); }
        if constexpr (LNS && QKV && SHADOW) f(a.n_raw);
        if constexpr (RS) f(a.stat_tiles);
        if constexpr (QKV) f(a.n_heads);
        if constexpr (QKV || CKV) { f(a.kv_fp8); f(a.head_dim); f(a.d_model); }
    }
};

// One output tile (column tile bx, row tile by) of the product described by st and tail.
// WNT: W is loaded with the non-temporal hint (GemmArgs::w_nt)
// NB: 64-wide k blocks per wavefront, K = 64 NW NB, known at compile time; 0: any K.  NW: wavefronts
//
// What bounds a launch at decode batches is latency: 8 MB of weights stream in 1.5 us behind the first HBM access, so
// every further round trip to memory shows.  Therefore
//  * everything a workgroup reads -- the first blocks of both operands, then row statistics, vectors, residual tile,
//    cache slots -- is requested before anything is waited for.  The memory counter is in order and a load behind a
//    branch makes the compiler wait for all loads before it, so no load sits behind one: indices are clamped instead
//    (buffers of fragment order are padded to whole tiles), null operands are read from W and replaced by zero;
//  * with NB known the k loop is straight-line code and each block is waited for on its own; with a run-time k loop
//    around conditional loads the compiler waited for the blocks just requested.
template <typename T, int PRO, int EPI, int MT, int NT, bool WNT, int NB, int NW = 4>
__device__ __forceinline__ void gemm_decode_body(const GemmStart& st, TailPtr tail, const int bx, const int by) {
    TailLoad<GemmFields<T, PRO, EPI>, GemmArgs> rest(tail);
    GemmArgs a;
    constexpr int BM = 16 * MT, BN = 16 * NT;
    constexpr int EP = (MT * NT + NW - 1) / NW;  // output 4-vectors per thread in the epilogue
    constexpr int ES = sizeof(T);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int m0 = by * BM, n0 = bx * BN;
    const int K = NB > 0 ? NB * NW * 64 : st.K, M = st.M;
    static_assert(NW == 4 || NB > 0, "more wavefronts: known K");
    const int nblk = K >> 8;  // 64-wide k blocks per wavefront
    const char* __restrict__ W = static_cast<const char*>(st.W);
    const char* __restrict__ A = static_cast<const char*>(st.A);

    constexpr bool LNS = PRO == PRO_LNS;         // LayerNorm around the product (see kernels.h):
    constexpr bool SHADOW = LNS && ES == 2;      // of the rows' shadow, corrected behind the product
    constexpr bool CENTRE = LNS && ES == 4;      // of the rows themselves, their mean taken off in front of it
    constexpr bool RS = EPI == EPI_RESID_S;      // residual update that also writes statistics (bfloat16: and shadow)

    __shared__ f32x4 part[NW][MT * NT][64];
    __shared__ float red[2][BM];  // LNS: the rows' means, the factors their products are scaled with

    // float32: either half of every block's products has its own sum.  A float32 decoder's error is made of the roundings along
    // such sums, and two of half the length have fewer large ones (relative error of the logits against float64, LayerNorm and one
    // sum / this: 4 layers of d_model 1024 4.07e-7 / 3.01e-7, 2 of 256 1.59e-7 / 1.31e-7).
    constexpr int SUMS = ES == 4 ? 2 : 1;
    f32x4 acc[SUMS][MT][NT];
#pragma unroll
    for (int i = 0; i < SUMS; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[i][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // block (n tile, k block i*4 + wave) of the re-ordered weights
    auto wblk = [&](int nt, int i) {
        return reinterpret_cast<const T*>(W + frag_block_off<ES>((n0 >> 4) + nt, i * NW + wave, K));
    };

    // ---- the operand stream: ring of D blocks in registers
    constexpr int D0 = (MT + NT) <= 2 ? 8 : (MT + NT) <= 4 ? 4 : 2;
    constexpr int DMAX = ES == 4 && D0 > 2 ? D0 / 2 : D0;
    constexpr int D = NB > 0 && NB < DMAX ? NB : DMAX;
    Frag16<T> af[D][MT], wf[D][NT];
    // 16-row tiles: A through a buffer descriptor; the lanes of rows from M on ask beyond its end and get zeros without a
    // request.  One row, 24 layers: 97.5 -> 95.3 ms for three utterances of 40 tokens.  Larger tiles have few such rows.
    const FragRows<ES> rows(A + frag_block_off<ES>(m0 >> 4, 0, K), M - m0, lane);
    auto fetch_w = [&](int slot, int i) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wf[slot][nt] = WNT ? load_frag_nt(wblk(nt, i), lane) : load_frag(wblk(nt, i), lane);
    };
    auto fetch_a = [&](int slot, int i) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if constexpr (MT == 1) rows.load(i * NW + wave, af[slot][mt]);
            else af[slot][mt] = load_frag(reinterpret_cast<const T*>(A + frag_block_off<ES>((m0 >> 4) + mt, i * NW + wave, K)), lane);
        }
    };
    auto fetch = [&](int slot, int i) {
        fetch_w(slot, i);
        fetch_a(slot, i);
    };
    float mean[MT];  // CENTRE: of this lane's row of every tile (RMSNorm: 0)
    auto compute = [&](int slot) {
        if constexpr (CENTRE && NB > 0 && MT * NT <= 2) {
            // The two sums in turn, and what a multiplication takes subtracted beside the ones before: left to itself the compiler puts
            // all multiplications of a sum one behind the other, each behind its own subtraction.  4 layers of d_model 1024, us a step
            // without it and the barrier behind fetch_stats / with both: 16 rows 191.8 / 187.8, 32 208.5 / 203.5, 64 243.2 / 240.4,
            // 128 353.9 / 356.9; on the larger tiles 1 to 2 % slower.
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int i = (k & 1) * 8 + (k >> 1);
                float v[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) v[mt] = af[slot][mt].v[i] - mean[mt];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        f32x4& sum = acc[i / 8][mt][nt];
                        sum = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[slot][nt].v[i], v[mt], sum, 0, 0, 0);
                    }
            }
            __builtin_amdgcn_sched_group_barrier(0x2, 2 * MT, 0);
#pragma unroll
            for (int k = 0; k < 14; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x8, MT * NT, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, MT, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x8, 2 * MT * NT, 0);
            return;
        }
        if constexpr (CENTRE) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) af[slot][mt].v[i] -= mean[mt];
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if constexpr (ES == 4) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        f32x4& sum = acc[i / 8][mt][nt];
                        sum = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[slot][nt].v[i], af[slot][mt].v[i], sum, 0, 0, 0);
                    }
                } else {
                    mma(acc[0][mt][nt], wf[slot][nt], af[slot][mt]);
                }
            }
    };
    // LNS: tile statistics of the rows being multiplied, 16 lanes per row, four 16-column tiles per lane.  Of 16 rows they
    // are requested in front of the stream and combined while it is on its way (4.13 -> 3.96 us for the QKV product of one
    // row); of more rows they would hold it back (8.2 -> 8.9 us at 256 rows) and are requested behind its first blocks.
    // CENTRE: the first multiplication waits for them, so they are in front of the stream always (4 layers of d_model 1024, us a step
    // with them behind its first blocks / in front: 128 rows 359.3 / 349.5, 300 784.2 / 773.4).
    constexpr int SR = 4 * NW, SP = LNS ? (BM + SR - 1) / SR : 1;  // rows a pass, passes
    constexpr bool ST_FIRST = MT == 1 || CENTRE;
    f32x4 sv[SP][2];
    auto fetch_stats = [&]() {
#pragma unroll
        for (int p = 0; p < SP; ++p) {
            const f32x4* sp = reinterpret_cast<const f32x4*>(st.stats_in + (size_t)(m0 + min(SR * p + (tid >> 4), BM - 1)) * st.stat_tiles +
                                                             min(4 * (tid & 15), st.stat_tiles - 4));
            sv[p][0] = sp[0];
            sv[p][1] = sp[1];
        }
    };
    auto combine_stats = [&]() {
#pragma unroll
        for (int p = 0; p < SP; ++p) {
            float2 rs = combine_tile_stats<CENTRE>(sv[p][0], sv[p][1], 4 * (tid & 15) < st.stat_tiles, st.stat_tiles);
            const float rstd = fold_norm(a.rms, (float)K, a.ln_eps, rs.y, rs.x);
            const int row = SR * p + (tid >> 4);
            if ((tid & 15) == 0 && row < BM) {
                red[0][row] = rs.x;
                red[1][row] = rstd;
            }
        }
    };
    if constexpr (LNS && ST_FIRST) fetch_stats();
    if constexpr (CENTRE && NB > 0 && MT * NT <= 2) {
        // Every wavefront waits for the statistics that the others fetch: those of all go ahead of anyone's stream.
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier");
        __builtin_amdgcn_sched_barrier(0);
    }
    // Weights that come from memory (WNT): those of all blocks of the ring first, then the rows, which come from the caches.  A
    // CU takes a request of 1 KB every 16 cycles, so the last of 32 leaves 0.8 us after the first; with weights and rows taking
    // turns the weights' longer trip began that much later.  24 layers: batch 64, 131 positions 133.0 -> 129.9 ms; batch 16,
    // 24 positions 26.3 -> 25.7; batch 128, 33 positions 44.5 -> 44.2.  Where the weights come from the caches too, taking
    // turns is faster, because the first block is complete sooner (4 layers, 43 positions: batch 1 17.4 ms, 17.7 with the
    // weights first; batch 64 7.42, 7.52).
    auto start_ring = [&]() {
        if constexpr (WNT) {
#pragma unroll
            for (int u = 0; u < D; ++u) fetch_w(u, u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < D; ++u) fetch_a(u, u);
        } else {
#pragma unroll
            for (int u = 0; u < D; ++u) fetch(u, u);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- epilogue operands (they do not depend on the product), requested behind the stream's first blocks
    const T* __restrict__ bias = nullptr;
    // columns from n_raw on are not normalised here (n_raw is a multiple of every tile width: uniform)
    bool raw = false;
    // kept as loaded (null bias / addend: whatever W holds there) until the epilogue uses them: a conversion or a select
    // here would wait for everything requested so far
    f32x4 e_bias[EP], e_res[EP], e_aux[EP];  // e_aux: c1 (SHADOW)
    typename Raw4<T>::type e_rbias[EP];      // not LNS
    float e_mu[EP];                          // SHADOW: the shift this row's shadow was written with; RS: the row's
                                             // mean before the update = the shift its new shadow is written with
    int e_slot[EP];                          // EPI_QKV: cache slot of the row; EPI_CROSSKV: its frame
    auto tile_row = [&](int t, int l) { return m0 + (t / NT) * 16 + (l & 15); };
    auto tile_col = [&](int t, int l) { return n0 + (t % NT) * 16 + (l >> 4) * 4; };
    auto request_epilogue = [&]() {
        rest.get(a);
        bias = static_cast<const T*>(a.bias);
        if constexpr (SHADOW && EPI == EPI_QKV) raw = a.n_raw > 0 && n0 >= a.n_raw;
#pragma unroll
        for (int j = 0; j < EP; ++j) {
            const int t = MT * NT < NW ? min(wave, MT * NT - 1) : wave + NW * j;
            const int m = tile_row(t, lane), n = tile_col(t, lane), mc = min(m, M - 1);
            if constexpr (LNS) {
                const float* c2 = a.ln_c2 + n;
                if constexpr (SHADOW && EPI == EPI_QKV) c2 = raw ? a.raw_bias + (n - a.n_raw) : c2;
                e_bias[j] = load_global<f32x4>(c2);
                if constexpr (SHADOW) {
                    int n_c1 = n;
                    if constexpr (EPI == EPI_QKV) n_c1 = raw ? n - a.n_raw : n;
                    e_aux[j] = *reinterpret_cast<const f32x4*>(a.ln_c1 + n_c1);
                }
            } else {
                e_rbias[j] = load_global<typename Raw4<T>::type>(bias ? static_cast<const void*>(bias + n) : W);
            }
            if constexpr ((LNS || RS) && ES == 2) e_mu[j] = a.mu_hat_in[m];
            if constexpr (RS) e_res[j] = *reinterpret_cast<const f32x4*>(static_cast<const char*>(a.out) + frag_elem_off<4>(m, n, a.N));
            if constexpr (EPI == EPI_F32 && PRO == PRO_T)  // optional addend, float [M,N] row-major like the output
                e_res[j] = load_global<f32x4>(a.addend ? static_cast<const void*>(a.addend + (size_t)mc * a.N + n) : W);
            if constexpr (EPI == EPI_QKV) e_slot[j] = a.kv_slot[mc];
            if constexpr (EPI == EPI_CROSSKV) e_slot[j] = load_global<int>(a.out_row_map ? static_cast<const void*>(a.out_row_map + mc) : W);
        }
        if constexpr (LNS && !ST_FIRST) fetch_stats();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LNS && ST_FIRST) combine_stats();
        if constexpr (CENTRE) {
            lds_barrier();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) mean[mt] = red[0][mt * 16 + (lane & 15)];
        }
    };

    if constexpr (NB > 0) {
        start_ring();
        request_epilogue();
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            compute(i % D);
            if (i + D < NB) fetch(i % D, i + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else if (nblk >= D) {
        start_ring();
        request_epilogue();
        int b0 = 0;
        for (; b0 + 2 * D <= nblk; b0 += D)
#pragma unroll
            for (int u = 0; u < D; ++u) {
                compute(u);
                fetch(u, b0 + D + u);
            }
        const int rem = nblk - b0;  // the ring holds the next min(rem, D) blocks; rem < 2 D
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < rem) {
                compute(u);
                if (D + u < rem) fetch(u, b0 + D + u);
            }
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (D + u < rem) compute(u);
    } else {
        // Fewer blocks than the ring holds (K = 256 on 16 x 16 tiles: one of eight).  Apart from the loop above: where a path
        // with fewer loads joins it, its waits are for the whole ring.  With the missing blocks fetched as copies of the last
        // one, a 6-layer decoder of d_model 256 at batch 300 took 9.38 ms for 35 positions, now 8.13; at batch 1 5.37, 4.87.
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < nblk) fetch(u, u);
        __builtin_amdgcn_sched_barrier(0);
        request_epilogue();
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < nblk) compute(u);
    }

    if constexpr (LNS && !ST_FIRST) combine_stats();
    // ---- sum the wavefronts' partial tiles in a fixed order, then the epilogue ----
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) part[wave][mt * NT + nt][lane] = SUMS == 2 ? acc[0][mt][nt] + acc[SUMS - 1][mt][nt] : acc[0][mt][nt];
    __syncthreads();

#pragma unroll
    for (int j = 0; j < EP; ++j) {
        const int t = wave + NW * j, l = lane;
        if (MT * NT < NW && t >= MT * NT) continue;
        f32x4 s = part[0][t][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += part[w][t][l];
        const int m = tile_row(t, l), n = tile_col(t, l);
        if (m >= M) continue;
        if constexpr (!LNS) {
            const f32x4 b = raw4_f32(e_rbias[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) e_bias[j][e] = bias ? b[e] : 0.f;
        }
        if constexpr (EPI == EPI_CROSSKV) e_slot[j] = a.out_row_map ? e_slot[j] : m;
        if constexpr (LNS) {
            const int rl = m - m0;
            const float mu = red[0][rl], rstd = red[1][rl];
            if constexpr (SHADOW && EPI == EPI_QKV)
                if (raw) {
                    // a product that belongs to a later normalisation of these rows (kernels.h, "merged products"):
                    // the bare sums (plus raw_bias) go to out2, whoever reads them finishes them
                    store4(a.out2 + (size_t)m * (a.N - a.n_raw) + (n - a.n_raw), s + e_bias[j]);
                    continue;
                }
            if constexpr (SHADOW) s -= (mu - e_mu[j]) * e_aux[j];
            s = s * rstd + e_bias[j];
            gemm_epilogue<T, EPI>(a, m, n, s, e_slot[j]);
            if constexpr (SHADOW)
                if (n == 0 && a.mu_hat_out) a.mu_hat_out[m] = mu;  // the layer's residual updates shift their shadows by this
        } else if constexpr (RS) {
            f32x4 x;
            if constexpr (ES == 4) x = e_res[j] + (s + e_bias[j]);  // one rounding at the size of the row, not two
            else x = e_res[j] + s + e_bias[j];
            *reinterpret_cast<f32x4*>(static_cast<char*>(a.out) + frag_elem_off<4>(m, n, a.N)) = x;
            if constexpr (ES == 2) store4(reinterpret_cast<T*>(static_cast<char*>(a.shadow_out) + frag_elem_off<ES>(m, n, a.N)), x - e_mu[j]);
            // this row's 16 columns of the tile sit in the four lanes l, l ^ 16, l ^ 32, l ^ 48
            const float tmean = rows4_sum((x[0] + x[1]) + (x[2] + x[3])) * (1.f / 16.f);
            const f32x4 dv = x - tmean;
            const float q = rows4_sum((dv[0] * dv[0] + dv[1] * dv[1]) + (dv[2] * dv[2] + dv[3] * dv[3]));
            if ((l >> 4) == 0) a.stats_out[(size_t)m * a.stat_tiles + (n >> 4)] = float2{tmean, q};
        } else {
            s += e_bias[j];
            if constexpr (EPI == EPI_F32 && PRO == PRO_T) { if (a.addend) s += e_res[j]; }
            gemm_epilogue<T, EPI>(a, m, n, s, e_slot[j]);
        }
    }
}

template <typename T, int PRO, int EPI, int MT, int NT, bool WNT, int NB, int NW = 4>
__global__ __launch_bounds__(64 * NW) void gemm_decode_kernel(const void* W, const void* A, const float2* stats_in, int M, int K,
                                                              int stat_tiles, ArgTail) {
    gemm_decode_body<T, PRO, EPI, MT, NT, WNT, NB, NW>(
        GemmStart{W, A, stats_in, M, K, stat_tiles}, tail_of<decltype(gemm_decode_kernel<T, PRO, EPI, MT, NT, WNT, NB, NW>)>(), blockIdx.x, blockIdx.y);
}

// Two products of the same operand A in one launch: the workgroups of z = 0 are the tiles of a0 (a residual update,
// EPI_RESID_S), those of z = 1 the tiles of a1 (kernels.h, "merged products").  Neither reads what the other writes.
template <typename T, int MT, int NT, int EPI1, bool WNT, int NB, int NW = 4>
__global__ __launch_bounds__(64 * NW) void gemm_decode_pair_kernel(const void* W0, const void* W1, const void* A, int M, int K,
                                                               ArgTail, ArgTail) {
    typedef decltype(gemm_decode_pair_kernel<T, MT, NT, EPI1, WNT, NB, NW>) Self;
    if (blockIdx.z == 0)
        gemm_decode_body<T, PRO_T, EPI_RESID_S, MT, NT, WNT, NB, NW>(GemmStart{W0, A, nullptr, M, K, 0}, tail_of<Self, 0>(), blockIdx.x, blockIdx.y);
    else
        gemm_decode_body<T, PRO_T, EPI1, MT, NT, WNT, NB, NW>(GemmStart{W1, A, nullptr, M, K, 0}, tail_of<Self, 1>(), blockIdx.x, blockIdx.y);
}

// The non-temporal hint for W (GemmArgs::w_nt) goes with launches of one workgroup per CU in at most four row tiles: the
// workgroups that share a panel of W then ask for it at the same time, later ones find nothing left of it in L2.  24 layers,
// 24 positions, ms without the hint / with it everywhere / by this rule: batch 64 25.6, 24.1, 24.1; 128 34.9, 33.3, 33.4; 160
// 39.3, 41.3, 39.1; 250 44.5 each.
constexpr long kCus = 256;  // compute units of an unpartitioned MI355X; the rules here are measured on one
static bool hint_w(const GemmArgs& a, long wgs, int row_tiles) { return a.w_nt && wgs <= kCus && row_tiles <= 4; }

// Dynamic LDS that keeps a second workgroup of the float32 32 x 32, 32 x 64 and 64 x 32 tiles off a CU (16 to 34 KB of 160
// are their own).  By registers two or three fit, and then each runs at less than half its speed: 528 rows, N = 4096,
// K = 1024 on 32 x 32 tiles 69.3 us shared, 55.4 alone; 64 x 32: 77.9, 57.8; N = 1024, K = 4096 on 32 x 32: 67.3, 51.9.  A
// launch of one round does not need it (130 rows, K = 4096: 17.9 us without, 19.0 with).
constexpr unsigned kOneWgLds = 66 << 10;

// Eight wavefronts a workgroup instead of four, of bfloat16 products over K = 1024 (nb = 4 blocks a wavefront) or 4096 (16):
// tiles of 512 outputs and more, and over 4096 the smallest, up to a workgroup a CU; 64 x 64 over 1024 always (one fits a CU either
// way).  Their operands are under way sooner, and a wavefront has half the matrix instructions behind them.  us a launch, four /
// eight wavefronts (weights of 24 layers in turn): N = 4096, K = 1024 on 32 x 64, 80 to 128 rows 4.42 to 4.53 / 4.18 to 4.29, from
// memory with the hint on 64 x 32 5.99 / 5.28; on 64 x 64, 256 rows 6.43 / 5.88, 512 10.98 / 10.00; N = 1024 on 32 x 64, 512 rows 4.58 /
// 4.43, on 64 x 64, 1024 rows 6.58 / 6.20; N = 1024, K = 4096 on 16 x 16, 64 rows 4.53 / 4.38 (24 layers, batch 64, 131 positions 124.1 ->
// 122.9 ms), on 32 x 16, 128 rows 5.60 / 5.50, from memory 7.50 / 7.27.  But 16 x 16 to 32 x 32 over 1024 4 to 8 % slower, 32 x 32 over 4096 1 %
// slower, 64 x 64 over 4096, 1024 rows 15.4 / 15.6; sixteen nowhere faster; 32 x 64, 256 rows, two a CU 6.42 / 6.92.
constexpr bool eight_wavefronts(int tiles, int nb) { return (nb == 4 && tiles >= 8) || (nb == 16 && (tiles <= 2 || tiles == 8)); }
constexpr bool always_eight(int tiles, int nb) { return nb == 4 && tiles == 16; }

template <typename T, int PRO, int EPI, int MT, int NT, int NB>
static hipError_t launch_nb(const GemmArgs& a, hipStream_t s) {
    dim3 grid(a.N / (16 * NT), (a.M + 16 * MT - 1) / (16 * MT));
    const long wgs = (long)grid.x * grid.y;
    const ArgTail tail = make_tail<GemmFields<T, PRO, EPI>>(a);
    unsigned lds = 0;
    // Where one workgroup has a CU to itself, eight wavefronts have its operands under way sooner than four.
    if constexpr (sizeof(T) == 2 && eight_wavefronts(MT * NT, NB)) {
        if (wgs <= kCus || always_eight(MT * NT, NB)) {
            if (hint_w(a, wgs, grid.y)) hipLaunchKernelGGL((gemm_decode_kernel<T, PRO, EPI, MT, NT, true, NB / 2, 8>), grid, dim3(512), 0, s, a.W, a.A, a.stats_in, a.M, a.K, a.stat_tiles, tail);
            else hipLaunchKernelGGL((gemm_decode_kernel<T, PRO, EPI, MT, NT, false, NB / 2, 8>), grid, dim3(512), 0, s, a.W, a.A, a.stats_in, a.M, a.K, a.stat_tiles, tail);
            return hipGetLastError();
        }
    }
    if constexpr (!(sizeof(T) == 2 && always_eight(MT * NT, NB))) {
    if constexpr (sizeof(T) == 4 && MT * NT >= 4 && MT * NT <= 8) {
        if (wgs > kCus) {
            static DeviceOnce once;
            hipError_t e = once.run([] {
                return hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_decode_kernel<T, PRO, EPI, MT, NT, false, NB>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kOneWgLds);
            });
            if (e != hipSuccess) return e;
            lds = kOneWgLds;
        }
    }
    if constexpr (sizeof(T) == 2) {  // float32 W is loaded the same way in both
        if (hint_w(a, wgs, grid.y)) {
            hipLaunchKernelGGL((gemm_decode_kernel<T, PRO, EPI, MT, NT, true, NB>), grid, dim3(256), 0, s, a.W, a.A, a.stats_in, a.M, a.K, a.stat_tiles, tail);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((gemm_decode_kernel<T, PRO, EPI, MT, NT, false, NB>), grid, dim3(256), lds, s, a.W, a.A, a.stats_in, a.M, a.K, a.stat_tiles, tail);
    }
    return hipGetLastError();
}
// K = 1024 and, for the second FFN product, K = 4096 are unrolled; every other K runs the loop
template <typename T, int PRO, int EPI, int MT, int NT>
static hipError_t launch_one(const GemmArgs& a, hipStream_t s) {
    if (a.K == 1024) return launch_nb<T, PRO, EPI, MT, NT, 4>(a, s);
    if constexpr (EPI == EPI_RESID_S)
        if (a.K == 4096) return launch_nb<T, PRO, EPI, MT, NT, 16>(a, s);
    return launch_nb<T, PRO, EPI, MT, NT, 0>(a, s);
}

// Tile choice: the candidate with the least cost per CU, then the fewest workgroups.  n_out: output columns of the whole
// launch.
//
// bfloat16: a traffic model.  Each workgroup pulls (BM * bytes(A) + BN * bytes(W)) * K through its CU and the launch's
// workgroups are spread over the 256 CUs.  W mostly comes from memory, A from the caches; the folded LayerNorm reads 512
// bytes of statistics per row of 2 KB.  Workgroups of the smaller tiles share a CU (two or three fit by registers), so
// beyond 256 workgroups the bytes through a CU grow in proportion, not in whole rounds.  The 64 x 64 tile runs one workgroup
// per CU; up to a workgroup a CU, on eight wavefronts, it costs less than its bytes say (K = 1024, N = 4096, us on 32 x 64 / 64 x 64: 160
// rows 5.92 / 5.63, 256 6.42 / 5.88; N = 1024, 700 rows 5.98 / 5.63), in several rounds half more (320 rows 7.98 and over 8.93, 700 13.6 /
// 14.5); over K = 4096 the start-up is a smaller part and the bytes decide (1024 rows 17.9 / 15.4).  The wider
// tile reads a weight panel more often: where weights come from memory, 64 x 32 is better than 32 x 64 (N = 4096, 128 rows 5.31 / 5.59,
// from the caches 4.62 / 4.29).
//
// float32: whole rounds of 256 workgroups, because workgroups that share a CU gain little or lose (kOneWgLds).  A round
// costs per k the larger of the matrix instructions (BM * BN at 154 TFLOP/s) and what the CU takes in, and 2.5 us of
// start-up.  Measured at K = 1024 / 4096, us a round: 16 x 16 2.8 / 7.5, 32 x 16 4.2 / 10.3, 32 x 32 6.4 / 17.5, 32 x 64 and
// 64 x 32 11 / 33.5, 64 x 64 19.5 / 65.
// Over 9 row counts from 65 to 1000 and the seven products of a 4-layer decoder (d_model 1024, FFN 4096, the cross K/V
// product on four times the rows) this choice is on average 0.6 % slower than the fastest tile and nowhere more than 6 %;
// choosing by bytes among all tiles was 20 % slower (130 rows: cross-attention query 15.0 us on 32 x 16, 10.2 on 32 x 32; FFN1
// 35.0 on 32 x 64, 24.1 on 64 x 64; FFN2 27.1 on 32 x 16, 17.9 on 32 x 32).
enum TileId { T11, T21, T22, T24, T42, T44 };
template <typename T, int PRO>
static TileId choose_tile(const GemmArgs& a, int n_out) {
    struct Cand { int mt, nt; };
    static const Cand cands[] = {{1, 1}, {2, 1}, {2, 2}, {2, 4}, {4, 2}, {4, 4}};
    const double a_bytes = PRO == PRO_LNS ? 1.25 * sizeof(T) : sizeof(T), w_bytes = 1.15 * sizeof(T);
    int best = 0;
    double best_cost = 1e300;
    long best_wgs = 0;
    for (int c = 0; c < 6; ++c) {
        const int bm = 16 * cands[c].mt, bn = 16 * cands[c].nt;
        if (a.N % bn != 0 || (cands[c].mt == 1 && a.K > FragRows<sizeof(T)>::kMaxK)) continue;
        const long wgs = (long)((a.M + bm - 1) / bm) * (n_out / bn);
        double cost;
        if constexpr (sizeof(T) == 4) {
            const double rounds = (double)((wgs + kCus - 1) / kCus);
            cost = rounds * ((double)a.K * std::max(bm * bn, 14 * (bm + bn)) + 450.0 * 1024);
        } else {
            const double rounds = wgs > kCus ? (double)wgs / kCus : 1.0;
            double factor = 1.0;
            if (c == T44 && a.K < 4096) factor = a.K == 1024 && wgs <= kCus ? 0.92 : 1.6;
            if (c == T24 && hint_w(a, wgs, (a.M + bm - 1) / bm)) factor = 1.05;
            cost = rounds * (bm * a_bytes + bn * w_bytes) * factor;
        }
        if (cost < best_cost || (cost == best_cost && wgs < best_wgs)) { best = c; best_cost = cost; best_wgs = wgs; }
    }
    return (TileId)best;
}

template <typename T, int PRO, int EPI>
static hipError_t launch_tiles(const GemmArgs& a, hipStream_t s) {
    const TileId best = choose_tile<T, PRO>(a, a.N);
    if (best == T11) return launch_one<T, PRO, EPI, 1, 1>(a, s);
    if (best == T22) return launch_one<T, PRO, EPI, 2, 2>(a, s);
    if (best == T21) return launch_one<T, PRO, EPI, 2, 1>(a, s);
    if (best == T24) return launch_one<T, PRO, EPI, 2, 4>(a, s);
    if (best == T42) return launch_one<T, PRO, EPI, 4, 2>(a, s);
    return launch_one<T, PRO, EPI, 4, 4>(a, s);
}

// The LDS-tiled kernel (bf16, 128 x 128 tiles, one workgroup a CU) takes as long for a few tiles as for 256 of them (K = 1024:
// 14 to 15 us a round), the streaming kernel's time goes with the rows: the first is faster where its rounds are full to
// more than 5/6.  K = 1024, us tiled / streamed: N = 4096, 700 rows (192 tiles) 14.4 / 13.7, 896 (224) 14.6 / 15.7, 1024 (256) 14.9 / 17.5,
// 1536 (384) 26.6 / 25.1, 2048 (512) 28.0 / 32.2; N = 3072, 1024 rows (192) 15.8 / 15.1, 2048 (384) 30.1 / 27.4, 3072 (576) 43.8 / 39.1.
// Over another K the streaming kernel loops and is slower: from 160 tiles on.
constexpr int kTiledMinTiles = 160;
static bool use_tiled(const GemmArgs& a) {
    if (a.N % 128 != 0) return false;
    const long tiles = (long)((a.M + 127) / 128) * (a.N / 128), rounds = (tiles + kCus - 1) / kCus;
    return a.K == 1024 ? 6 * tiles > 5 * kCus * rounds : tiles >= kTiledMinTiles;
}

// The 256 x 256 direct-to-LDS kernel (cross K/V product only) needs whole 256-row tiles in A and enough
// tiles to occupy most of the compute units with one workgroup each.
constexpr int kDmaMinTiles = 160;
static bool use_dma_crosskv(const GemmArgs& a) {
    return a.N % 256 == 0 && a.N == 2 * a.d_model && a.K >= 256 &&
           a.a_rows >= (a.M + 255) / 256 * 256 && (long)((a.M + 255) / 256) * (a.N / 256) >= kDmaMinTiles;
}

// The row statistics behind a folded LayerNorm: 16 lanes share a row of at most 64 tiles (d_model <= 1024)
static bool stat_tiles_ok(int n) { return n >= 4 && n % 4 == 0 && n <= 64; }

template <typename T> static hipError_t launch_typed(GemmPro pro, GemmEpi epi, const GemmArgs& a, hipStream_t s) {
    constexpr bool tiled = sizeof(T) == 2;  // the kernels with operands in LDS take bfloat16
    if (pro == PRO_LNS) {
        if (!a.stats_in || !a.ln_c2 || (tiled && (!a.mu_hat_in || !a.ln_c1)) || !stat_tiles_ok(a.stat_tiles)) return hipErrorInvalidValue;
        if (epi == EPI_QKV && !a.kv_slot) return hipErrorInvalidValue;
        if (tiled && use_tiled(a)) return launch_gemm_tiled(epi, a, s);
        if (epi == EPI_QKV) return launch_tiles<T, PRO_LNS, EPI_QKV>(a, s);
        if (epi == EPI_F32) return launch_tiles<T, PRO_LNS, EPI_F32>(a, s);
        if (epi == EPI_RELU_T) return launch_tiles<T, PRO_LNS, EPI_RELU_T>(a, s);
    }
    if (pro == PRO_T && epi == EPI_RESID_S) {
        if (!a.stats_out || (tiled && (!a.mu_hat_in || !a.shadow_out)) || !stat_tiles_ok(a.stat_tiles) || a.stat_tiles * 16 != a.N)
            return hipErrorInvalidValue;
        return launch_tiles<T, PRO_T, EPI_RESID_S>(a, s);
    }
    if (pro == PRO_T && epi == EPI_CROSSKV) {
        if (tiled && use_dma_crosskv(a)) return launch_gemm_dma_crosskv(a, s);
        if (tiled && use_tiled(a)) return launch_gemm_tiled(epi, a, s);
        return launch_tiles<T, PRO_T, EPI_CROSSKV>(a, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- two products in one launch
template <typename T, int MT, int NT, int EPI1, int NB>
static hipError_t launch_pair_nb(const GemmArgs& a0, const GemmArgs& a1, hipStream_t s) {
    const int rows = (a0.M + 16 * MT - 1) / (16 * MT);
    const dim3 grid(a0.N / (16 * NT), rows, 2);
    const long wgs = 2l * grid.x * rows;
    const ArgTail t0 = make_tail<GemmFields<T, PRO_T, EPI_RESID_S>>(a0), t1 = make_tail<GemmFields<T, PRO_T, EPI1>>(a1);
    if constexpr (eight_wavefronts(MT * NT, NB)) {
        if (wgs <= kCus) {
            if (hint_w(a0, wgs, rows))
                hipLaunchKernelGGL((gemm_decode_pair_kernel<T, MT, NT, EPI1, true, NB / 2, 8>), grid, dim3(512), 0, s, a0.W, a1.W, a0.A, a0.M, a0.K, t0, t1);
            else
                hipLaunchKernelGGL((gemm_decode_pair_kernel<T, MT, NT, EPI1, false, NB / 2, 8>), grid, dim3(512), 0, s, a0.W, a1.W, a0.A, a0.M, a0.K, t0, t1);
            return hipGetLastError();
        }
    }
    if (hint_w(a0, wgs, rows))
        hipLaunchKernelGGL((gemm_decode_pair_kernel<T, MT, NT, EPI1, true, NB>), grid, dim3(256), 0, s, a0.W, a1.W, a0.A, a0.M, a0.K, t0, t1);
    else
        hipLaunchKernelGGL((gemm_decode_pair_kernel<T, MT, NT, EPI1, false, NB>), grid, dim3(256), 0, s, a0.W, a1.W, a0.A, a0.M, a0.K, t0, t1);
    return hipGetLastError();
}
template <typename T, int EPI1, int NB>
static hipError_t launch_pair_tiles(const GemmArgs& a0, const GemmArgs& a1, hipStream_t s) {
    switch (choose_tile<T, PRO_T>(a0, a0.N + a1.N)) {  // the batches this is used for have at most 256 rows
        case T11: return launch_pair_nb<T, 1, 1, EPI1, NB>(a0, a1, s);
        case T21: return launch_pair_nb<T, 2, 1, EPI1, NB>(a0, a1, s);
        case T22: return launch_pair_nb<T, 2, 2, EPI1, NB>(a0, a1, s);
        default: return launch_pair_nb<T, 4, 2, EPI1, NB>(a0, a1, s);
    }
}

hipError_t launch_gemm_pair(Dtype dt, const GemmArgs& a0, GemmEpi epi1, const GemmArgs& a1, hipStream_t s) {
    if (dt != kBF16 || a0.M < 1 || a0.M != a1.M || a0.M > 256 || a0.K % 256 != 0 || a1.A != a0.A || a1.K != a0.K || a1.N != a0.N || a0.N % 32 != 0)
        return hipErrorInvalidValue;
    if (!a0.stats_out || !a0.mu_hat_in || !a0.shadow_out || !stat_tiles_ok(a0.stat_tiles) || a0.stat_tiles * 16 != a0.N)
        return hipErrorInvalidValue;
    if (epi1 == EPI_F32)
        return a0.K == 1024 ? launch_pair_tiles<bf16_t, EPI_F32, 4>(a0, a1, s) : launch_pair_tiles<bf16_t, EPI_F32, 0>(a0, a1, s);
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(Dtype dt, GemmPro pro, GemmEpi epi, const GemmArgs& a, hipStream_t s) {
    if (a.M < 1 || a.K % 256 != 0 || a.N % 64 != 0) return hipErrorInvalidValue;
    return dt == kBF16 ? launch_typed<bf16_t>(pro, epi, a, s) : launch_typed<float>(pro, epi, a, s);
}

// ---------------------------------------------------------------- LayerNorm folding (once, at create)
// One wavefront per output column: c1[n] = sum_k W[n,k] g[k] (c1 null: not wanted), c2[n] = sum_k W[n,k] b[k] + bias[n].
template <typename T>
__global__ __launch_bounds__(256) void fold_ln_kernel(const T* __restrict__ W, const T* __restrict__ g,
                                                      const T* __restrict__ b, const T* __restrict__ bias,
                                                      float* __restrict__ c1, float* __restrict__ c2, int N, int K) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n >= N) return;
    float s1 = 0.f, s2 = 0.f;
    for (int k = lane; k < K; k += 64) {
        const float w = (float)W[(size_t)n * K + k];
        s1 += to_f32(from_f32<T>(w * (float)g[k]));  // the column-scaled matrix as reorder_weight_kernel stores it
        if (b) s2 += w * (float)b[k];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s1 += __shfl_xor(s1, off);
        s2 += __shfl_xor(s2, off);
    }
    if (lane == 0) {
        if (c1) c1[n] = s1;
        c2[n] = s2 + (bias ? (float)bias[n] : 0.f);
    }
}

hipError_t launch_fold_ln(Dtype dt, const void* W, const void* g, const void* b, const void* bias, float* c1, float* c2,
                          int N, int K, hipStream_t s) {
    const dim3 grid((N + 3) / 4);
    if (dt == kBF16)
        hipLaunchKernelGGL(fold_ln_kernel<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t*>(W),
                           static_cast<const bf16_t*>(g), static_cast<const bf16_t*>(b),
                           static_cast<const bf16_t*>(bias), c1, c2, N, K);
    else
        hipLaunchKernelGGL(fold_ln_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(W),
                           static_cast<const float*>(g), static_cast<const float*>(b), static_cast<const float*>(bias),
                           c1, c2, N, K);
    return hipGetLastError();
}

// ---------------------------------------------------------------- weight re-ordering
// dst (fragment order) <- src (row-major [N, K]), columns scaled by gain (may be null); one thread per 16-byte piece.
template <typename T>
__global__ __launch_bounds__(256) void reorder_weight_kernel(const T* __restrict__ src, const T* __restrict__ gain,
                                                             char* __restrict__ dst, int N, int K, int dst_k0, int dst_K) {
    constexpr int ES = sizeof(T), EPP = 16 / ES;
    const size_t piece = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t n_pieces = (size_t)N * K / EPP;
    if (piece >= n_pieces) return;
    const int n = (int)(piece / (K / EPP));
    const int k = (int)(piece % (K / EPP)) * EPP;
    T v[EPP];
    *reinterpret_cast<f32x4*>(v) = *reinterpret_cast<const f32x4*>(src + (size_t)n * K + k);  // 16 bytes, any type
    if (gain) {
#pragma unroll
        for (int e = 0; e < EPP; ++e) v[e] = from_f32<T>(to_f32(v[e]) * to_f32(gain[k + e]));
    }
    *reinterpret_cast<f32x4*>(dst + frag_elem_off<ES>(n, dst_k0 + k, dst_K)) = *reinterpret_cast<const f32x4*>(v);
}

// Product of two weight matrices for a merged product (kernels.h): P[n, k] = sum_j T(W1[n, j] g[j]) W2[j, k], float32 sums
// of the stored (rounded) factors, rounded to T once and written in fragment order into columns dst_k0 .. dst_k0 + K
// of a matrix with dst_K columns.  W1 [N, J], W2 [J, K] row-major; g may be null.  One 64 x 64 output tile per
// workgroup, 4 x 4 outputs per thread, 16-deep slices through LDS.  Runs once, when the decoder is created.
template <typename T>
__global__ __launch_bounds__(256) void weight_product_kernel(const T* __restrict__ W1, const T* __restrict__ g,
                                                             const T* __restrict__ W2, char* __restrict__ dst, int N, int J,
                                                             int K, int dst_k0, int dst_K) {
    __shared__ float sa[16][64 + 4], sb[16][64 + 4];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int n0 = blockIdx.y * 64, k0 = blockIdx.x * 64;
    float acc[4][4] = {};
    for (int j0 = 0; j0 < J; j0 += 16) {
        for (int i = tid; i < 64 * 16; i += 256) {
            const int n = i >> 4, j = i & 15;  // W1 tile: 64 rows x 16 j, read along j
            float w = to_f32(W1[(size_t)(n0 + n) * J + j0 + j]);
            if (g) w = to_f32(from_f32<T>(w * to_f32(g[j0 + j])));
            sa[j][n] = w;
            const int jj = i >> 6, k = i & 63;  // W2 tile: 16 j x 64 columns, read along k
            sb[jj][k] = to_f32(W2[(size_t)(j0 + jj) * K + k0 + k]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            float av[4], bv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { av[u] = sa[j][ty * 4 + u]; bv[u] = sb[j][tx * 4 + u]; }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fmaf(av[u], bv[v], acc[u][v]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int n = n0 + ty * 4 + u, k = k0 + tx * 4;
        store4(reinterpret_cast<T*>(dst + frag_elem_off<sizeof(T)>(n, dst_k0 + k, dst_K)),
               f32x4{acc[u][0], acc[u][1], acc[u][2], acc[u][3]});
    }
}

hipError_t launch_weight_product(Dtype dt, const void* W1, const void* g, const void* W2, void* dst, int N, int J, int K,
                                 int dst_k0, int dst_K, hipStream_t s) {
    if (dt != kBF16 || N % 64 != 0 || K % 64 != 0 || J % 16 != 0 || dst_k0 % 64 != 0 || dst_K % 64 != 0 || dst_k0 + K > dst_K)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(weight_product_kernel<bf16_t>, dim3(K / 64, N / 64), dim3(256), 0, s, static_cast<const bf16_t*>(W1),
                       static_cast<const bf16_t*>(g), static_cast<const bf16_t*>(W2), static_cast<char*>(dst), N, J, K, dst_k0, dst_K);
    return hipGetLastError();
}

// out[n] = sum_j T(W[n, j] g[j]) v[j] (float32; v null: zeros).  One wavefront per n.
template <typename T>
__global__ __launch_bounds__(256) void fold_vec_kernel(const T* __restrict__ W, const T* __restrict__ g, const T* __restrict__ v,
                                                       float* __restrict__ out, int N, int J) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n >= N) return;
    float sum = 0.f;
    if (v)
        for (int j = lane; j < J; j += 64) {
            float w = to_f32(W[(size_t)n * J + j]);
            if (g) w = to_f32(from_f32<T>(w * to_f32(g[j])));
            sum += w * to_f32(v[j]);
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) out[n] = sum;
}

hipError_t launch_fold_vec(Dtype dt, const void* W, const void* g, const void* v, float* out, int N, int J, hipStream_t s) {
    if (dt != kBF16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fold_vec_kernel<bf16_t>, dim3((N + 3) / 4), dim3(256), 0, s, static_cast<const bf16_t*>(W),
                       static_cast<const bf16_t*>(g), static_cast<const bf16_t*>(v), out, N, J);
    return hipGetLastError();
}

// dst (fragment order, [M, K]) <- rows of a row-major source, row m taken from src row row_map[m] (or m).  A copy, bound
// by memory: a wavefront moves 16-row x 64-k blocks, lane (r, g) the 16 elements of row r that it would hold for the MFMA,
// so a block's loads take whole 128-byte lines of 16 rows and every store instruction writes 1 KB in one piece; all loads
// of four blocks are in flight before the first store.  (One workgroup per row, whose stores were 16-byte pieces 256 bytes
// apart, took 1272 us for 512 000 rows of 1024 bf16 = 1.65 TB/s and 120 us for 63 913 gathered rows.)
template <typename T>
__global__ __launch_bounds__(256) void reorder_rows_kernel(const T* __restrict__ src, const int* __restrict__ row_map,
                                                           char* __restrict__ dst, int M, int K) {
    constexpr int ES = sizeof(T);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nkb = K >> 6;
    const int m = blockIdx.x * 16 + (lane & 15);
    if (m >= M) return;
    const size_t srow = row_map ? (size_t)row_map[m] : (size_t)m;
    const T* p = src + srow * K + (lane >> 4) * 16;
    char* q = dst + frag_block_off<ES>(blockIdx.x, 0, K) + lane * 16;
    for (int k0 = wave; k0 < nkb; k0 += 16) {
        f32x4 v[4][ES];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T* s = p + (size_t)min(k0 + 4 * u, nkb - 1) * 64;
#pragma unroll
            for (int j = 0; j < ES; ++j) v[u][j] = reinterpret_cast<const f32x4*>(s)[j];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + 4 * u < nkb)
#pragma unroll
                for (int j = 0; j < ES; ++j)
                    *reinterpret_cast<f32x4*>(q + ((size_t)(k0 + 4 * u) * ES + j) * 1024) = v[u][j];
    }
}

hipError_t launch_reorder_rows(Dtype dt, const void* src, const int* row_map, void* dst, int M, int K, hipStream_t s) {
    if (M < 1 || K % 64 != 0) return hipErrorInvalidValue;
    if (dt == kBF16)
        hipLaunchKernelGGL(reorder_rows_kernel<bf16_t>, dim3((M + 15) / 16), dim3(256), 0, s, static_cast<const bf16_t*>(src), row_map,
                           static_cast<char*>(dst), M, K);
    else
        hipLaunchKernelGGL(reorder_rows_kernel<float>, dim3((M + 15) / 16), dim3(256), 0, s, static_cast<const float*>(src), row_map,
                           static_cast<char*>(dst), M, K);
    return hipGetLastError();
}

hipError_t launch_reorder_weight(Dtype dt, const void* src, const void* gain, void* dst, int N, int K, hipStream_t s,
                                 int dst_k0, int dst_K) {
    if (dst_K <= 0) dst_K = K;
    if (N % 16 != 0 || K % 64 != 0 || dst_k0 % 64 != 0 || dst_K % 64 != 0 || dst_k0 + K > dst_K) return hipErrorInvalidValue;
    const size_t pieces = (size_t)N * K / (dt == kBF16 ? 8 : 4);
    dim3 grid((unsigned)((pieces + 255) / 256));
    if (dt == kBF16)
        hipLaunchKernelGGL(reorder_weight_kernel<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t*>(src),
                           static_cast<const bf16_t*>(gain), static_cast<char*>(dst), N, K, dst_k0, dst_K);
    else
        hipLaunchKernelGGL(reorder_weight_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(src),
                           static_cast<const float*>(gain), static_cast<char*>(dst), N, K, dst_k0, dst_K);
    return hipGetLastError();
}

}  // namespace aed
