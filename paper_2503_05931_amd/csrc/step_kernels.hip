// Small kernels of the decoder step: token + position embedding, the greedy
// sampler with its device-side sequence state, and state bookkeeping.
//
// All per-sequence state that changes from step to step (position, number of
// generated tokens, finished flag, next input token) lives in device memory and
// is advanced by the sampler, so one captured launch graph can be replayed for
// every step without touching its arguments.
#include <limits.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace aed {

// where position pos of sequence b is cached: page * 16 + place in the page
__device__ __forceinline__ int slot_of(const StateArgs& st, int b, int pos) {
    return st.page_table[(size_t)b * st.max_pages + min(max(pos, 0) >> 4, st.max_pages - 1)] * kPage + (pos & (kPage - 1));
}

__device__ __forceinline__ int clamped(int v, int n) { return v < 0 ? 0 : v >= n ? n - 1 : v; }

// One row's embedding: the residual row and its tile statistics, with bfloat16 its shadow and shift.  Every
// thread of the workgroup; pv: the thread's elements of the position's row; slot: where the position is cached, -1: nowhere.
template <typename T>
__device__ __forceinline__ void embed_row(const EmbedArgs& ea, const StateArgs& st, int b, int tok, f32x4 pv, int slot) {
    const int tid = threadIdx.x, d = ea.d;
    const ShadowArgs& sh = ea.sh;
    if (tid == 0) st.kv_slot[b] = slot;
    const T* e = static_cast<const T*>(ea.tok_emb) + (size_t)clamped(tok, st.vocab) * d;
    const int i = tid * 4;  // d <= 1024: one 4-vector per thread
    const bool live = i < d;
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
    if (live) {
        const f32x4 ev = load4(e + i);
        o[0] = ea.emb_scale * ev[0] + pv[0];
        o[1] = ea.emb_scale * ev[1] + pv[1];
        o[2] = ea.emb_scale * ev[2] + pv[2];
        o[3] = ea.emb_scale * ev[3] + pv[3];
        store4(reinterpret_cast<float*>(reinterpret_cast<char*>(ea.x) + frag_elem_off<4>(b, i, d)), o);
    }
    float ts = (o[0] + o[1]) + (o[2] + o[3]);
    float mean = 0.f;  // RMSNorm: no shift
    if constexpr (sizeof(T) == 2) {  // row mean over the workgroup, for the shadow
        __shared__ float wsum[4];
        float s = ts;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if ((tid & 63) == 0) wsum[tid >> 6] = s;
        __syncthreads();
        if (!sh.rms) mean = (wsum[0] + wsum[1] + wsum[2] + wsum[3]) / (float)d;
    }
    // tile statistics over the 4 threads of a 16-column tile
    ts += __shfl_xor(ts, 1);
    ts += __shfl_xor(ts, 2);
    const float tmean = ts * (1.f / 16.f);
    float q = (o[0] - tmean) * (o[0] - tmean) + (o[1] - tmean) * (o[1] - tmean) + (o[2] - tmean) * (o[2] - tmean) +
              (o[3] - tmean) * (o[3] - tmean);
    q += __shfl_xor(q, 1);
    q += __shfl_xor(q, 2);
    if (!live) return;
    if ((tid & 3) == 0) sh.stats[(size_t)b * (d >> 4) + (i >> 4)] = float2{tmean, q};
    if constexpr (sizeof(T) == 2) {
        store4(reinterpret_cast<T*>(static_cast<char*>(sh.shadow) + frag_elem_off<2>(b, i, d)), o - mean);
        if (tid == 0) sh.mu_hat[b] = mean;
    }
}

// this thread's elements of a position's row
template <typename T> __device__ __forceinline__ f32x4 pos_row(const EmbedArgs& ea, int pos) {
    const int i = threadIdx.x * 4;
    if (i >= ea.d) return f32x4{0.f, 0.f, 0.f, 0.f};
    return load4(static_cast<const T*>(ea.pos_emb) + (size_t)min(pos, ea.max_positions - 1) * ea.d + i);
}

template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs ea, StateArgs st) {
    const int b = blockIdx.x, pos = st.seq_len[b];
    const int slot = slot_of(st, b, min(pos, ea.max_positions - 1));
    embed_row<T>(ea, st, b, st.cur_tok[b], pos_row<T>(ea, pos), st.finished[b] ? -1 : slot);
}

static bool embed_fits(const EmbedArgs& ea) { return ea.d <= 1024 && ea.d % 64 == 0; }

hipError_t launch_embed(Dtype dt, const EmbedArgs& ea, const StateArgs& st, hipStream_t s) {
    if (!embed_fits(ea)) return hipErrorInvalidValue;
    if (dt == kBF16) hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3(st.batch), dim3(256), 0, s, ea, st);
    else hipLaunchKernelGGL(embed_kernel<float>, dim3(st.batch), dim3(256), 0, s, ea, st);
    return hipGetLastError();
}

// argmax with the lowest index on ties: (value, index) pairs ordered by value
// descending, then index ascending.
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// What a sequence feeds next: token, position, and whether it is through.  The same in every thread of the workgroup.
struct Next { int tok, pos; bool through; };

// GREEDY: prompt feeding, EOS rules, output writes; else the argmax alone, into step_out (may be null) too.
// request(pos, fin): what else the caller reads that depends on the state words only, asked for behind the row's first loads
template <bool GREEDY, typename F>
__device__ __forceinline__ Next sample_row(const float* __restrict__ logits, const StateArgs& st, int* __restrict__ step_out,
                                           F request) {
    const int b = blockIdx.x, tid = threadIdx.x;
    // everything the decision needs is requested at once: the state words and this thread's share of the row
    // (vocab is a multiple of 64: 4-vectors; up to four per thread in flight, then the rest of a long row)
    const int fin = GREEDY ? st.finished[b] : 0;
    const int pos = st.seq_len[b];
    const int n = GREEDY ? st.n_gen[b] : 0;
    const int lim = GREEDY ? st.limit[b] : INT_MAX;
    const float* row = logits + (size_t)b * st.vocab;
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = tid * 4 + u * 1024;
        v[u] = i < st.vocab ? *reinterpret_cast<const f32x4*>(row + i) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    request(pos, fin);
    if (fin) return Next{st.cur_tok[b], pos, true};
    if (GREEDY && pos + 1 < st.prompt_len) {  // still feeding the prompt: no token is emitted
        const int fed = st.prompt[(size_t)b * st.prompt_stride + pos + 1];
        __syncthreads();  // every wavefront has read the position before it moves on
        if (tid == 0) {
            st.cur_tok[b] = fed;
            st.seq_len[b] = pos + 1;
        }
        return Next{fed, pos + 1, false};
    }
    float bv = -INFINITY;
    int bi = INT_MAX;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = tid * 4 + u * 1024 + e;
            if (i < st.vocab && better(v[u][e], i, bv, bi)) { bv = v[u][e]; bi = i; }
        }
    for (int base = tid * 4 + 4096; base < st.vocab; base += 1024) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(row + base);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (better(w[e], base + e, bv, bi)) { bv = w[e]; bi = base + e; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off);
        const int oi = __shfl_xor(bi, off);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    __shared__ float sv[4];
    __shared__ int si[4];
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
    __syncthreads();
    // every thread takes the decision, so that all of them know whether the sequence ends
    bv = sv[0];
    bi = si[0];
    for (int w = 1; w < 4; ++w)
        if (better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    int tok = bi == INT_MAX ? 0 : bi;
    if (!GREEDY) {
        const Next next{tok, pos + 1, false};
        if (tid != 0) return next;
        if (step_out) step_out[b] = tok;
        st.cur_tok[b] = tok;
        st.seq_len[b] = pos + 1;
        return next;
    }
    if (n + 1 >= lim) tok = st.eos_id;  // forced end at the per-sequence target length
    const bool ends = (st.eos_id >= 0 && tok == st.eos_id) || n + 1 >= st.max_new;
    if (ends)
        for (int i = tid; i < st.n_items; i += 256)
            if (st.items[i].x == b) st.items[i].x = b | kItemOff;
    const Next next{tok, pos + 1, ends};
    if (tid != 0) return next;
    st.out_tokens[(size_t)b * st.out_stride + n] = tok;
    st.n_gen[b] = n + 1;
    st.cur_tok[b] = tok;
    st.seq_len[b] = pos + 1;
    if (ends) {
        st.finished[b] = 1;
        atomicAdd(st.n_finished, 1);
    }
    return next;
}

__global__ __launch_bounds__(256) void sample_kernel(const float* __restrict__ logits, StateArgs st, int* __restrict__ step_out) {
    sample_row<false>(logits, st, step_out, [](int, int) {});
}

// The greedy step's last kernel: the sampler, then the embedding of what the sequence feeds next, so that a step begins
// with its first layer.  Both are one workgroup a sequence and nothing but a trip to memory each; the position's row and
// cache slot come with the logits, the token's row is the one trip more.
// Two layers of float32, batch 4, 32 tokens 2.43 -> 2.32 ms; 4 layers: batch 256, 128 tokens 41.45 -> 41.09, batch 203 with
// 8-bit caches, 64 tokens 16.75 -> 16.55, float32 batch 32, 32 tokens 10.42 -> 10.30.
template <typename T>
__global__ __launch_bounds__(256) void sample_embed_kernel(const float* __restrict__ logits, StateArgs st, EmbedArgs ea) {
    const int b = blockIdx.x;
    f32x4 pv;
    int slot;
    const Next next = sample_row<true>(logits, st, nullptr, [&](int pos, int fin) {
        const int at = fin ? pos : pos + 1;
        pv = pos_row<T>(ea, at);
        slot = slot_of(st, b, min(at, ea.max_positions - 1));
    });
    embed_row<T>(ea, st, b, next.tok, pv, next.through ? -1 : slot);
}

hipError_t launch_sample_embed(Dtype dt, const float* logits, const StateArgs& st, const EmbedArgs& ea, hipStream_t s) {
    if (!embed_fits(ea)) return hipErrorInvalidValue;
    if (dt == kBF16) hipLaunchKernelGGL(sample_embed_kernel<bf16_t>, dim3(st.batch), dim3(256), 0, s, logits, st, ea);
    else hipLaunchKernelGGL(sample_embed_kernel<float>, dim3(st.batch), dim3(256), 0, s, logits, st, ea);
    return hipGetLastError();
}

hipError_t launch_sample(const float* logits, const StateArgs& st, int* step_out, hipStream_t s) {
    hipLaunchKernelGGL(sample_kernel, dim3(st.batch), dim3(256), 0, s, logits, st, step_out);
    return hipGetLastError();
}

__global__ void reset_kernel(StateArgs st, const int* __restrict__ limits, int start_pos) {
    const int b = blockIdx.x;
    if (threadIdx.x == 0) {
        st.seq_len[b] = start_pos;
        st.n_gen[b] = 0;
        st.finished[b] = 0;
        st.cur_tok[b] = st.prompt[(size_t)b * st.prompt_stride + start_pos];
        st.limit[b] = limits ? limits[b] : INT_MAX;
        if (b == 0) *st.n_finished = 0;
    }
    for (int i = b * blockDim.x + threadIdx.x; i < st.n_items; i += gridDim.x * blockDim.x) st.items[i].x &= ~kItemOff;
    for (int t = threadIdx.x; t < st.max_new; t += blockDim.x) st.out_tokens[(size_t)b * st.out_stride + t] = st.pad_id;
}

hipError_t launch_reset(const StateArgs& st, const int* limits_dev, int start_pos, hipStream_t s) {
    hipLaunchKernelGGL(reset_kernel, dim3(st.batch), dim3(64), 0, s, st, limits_dev, start_pos);
    return hipGetLastError();
}

// A batch's start in one launch: the host's tables out of pinned memory into their places, the padded tensor's row map (65
// thousand entries built on the host and uploaded kept the GPU waiting), arrival counters and sequence state cleared.  As two
// uploads, a memset and two kernels the GPU waited 9 to 18 us in front of each.
__global__ __launch_bounds__(256) void start_batch_kernel(StartArgs a, StateArgs st) {
    const int b = blockIdx.x, tid = threadIdx.x, at = b * blockDim.x + tid, all = gridDim.x * blockDim.x;
    if (tid == 0) {
        st.seq_len[b] = 0;
        st.n_gen[b] = 0;
        st.finished[b] = 0;
        st.cur_tok[b] = 0;
        st.limit[b] = INT_MAX;
        if (b == 0) *st.n_finished = 0;
    }
    for (int i = at; i < st.n_items; i += all) st.items[i] = a.src_items[i];
    for (int i = at; i < a.n_counters; i += all) a.counters[i] = 0;
    if (a.row_map) {
        const int first = a.src_off[b], n = a.src_off[b + 1] - first;
        for (int t = tid; t < n; t += blockDim.x) a.row_map[first + t] = b * a.t_max + t;
    }
}

hipError_t launch_start_batch(const StartArgs& a, const StateArgs& st, hipStream_t s) {
    hipLaunchKernelGGL(start_batch_kernel, dim3(st.batch), dim3(256), 0, s, a, st);
    return hipGetLastError();
}

// A step's results to the caller's buffers: one launch where two copies were two, each with the GPU idle in front of it.
__global__ __launch_bounds__(256) void hand_out_kernel(const int* __restrict__ ids, int* __restrict__ ids_out, int batch,
                                                       const f32x4* __restrict__ logits, f32x4* __restrict__ logits_out, size_t n4) {
    const size_t at = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (ids_out)
        for (size_t i = at; i < (size_t)batch; i += (size_t)gridDim.x * 256) ids_out[i] = ids[i];
    if (logits_out)
        for (size_t i = at; i < n4; i += (size_t)gridDim.x * 256) logits_out[i] = logits[i];
}

hipError_t launch_hand_out(const int* ids, int* ids_out, int batch, const float* logits, float* logits_out, size_t n, hipStream_t s) {
    if (n % 4 != 0 || (uintptr_t)logits_out % 16 != 0) return hipErrorInvalidValue;
    const size_t blocks = std::min<size_t>(2048, ((logits_out ? n / 4 : batch) + 255) / 256);
    hipLaunchKernelGGL(hand_out_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ids, ids_out, batch, reinterpret_cast<const f32x4*>(logits),
                       reinterpret_cast<f32x4*>(logits_out), n / 4);
    return hipGetLastError();
}

__global__ void set_tokens_kernel(int* __restrict__ cur_tok, const int* __restrict__ src, int stride, int batch) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < batch) cur_tok[b] = src[(size_t)b * stride];
}

hipError_t launch_set_tokens(int* cur_tok, const int* src, int stride, int batch, hipStream_t s) {
    hipLaunchKernelGGL(set_tokens_kernel, dim3((batch + 255) / 256), dim3(256), 0, s, cur_tok, src, stride, batch);
    return hipGetLastError();
}

__global__ void copy_out_kernel(StateArgs st, int* __restrict__ dst_tokens, int* __restrict__ dst_lens) {
    const int b = blockIdx.x;
    for (int t = threadIdx.x; t < st.max_new; t += blockDim.x)
        dst_tokens[(size_t)b * st.max_new + t] = st.out_tokens[(size_t)b * st.out_stride + t];
    if (threadIdx.x == 0) dst_lens[b] = st.n_gen[b];
}

hipError_t launch_copy_out(const StateArgs& st, int* dst_tokens, int* dst_lens, hipStream_t s) {
    hipLaunchKernelGGL(copy_out_kernel, dim3(st.batch), dim3(64), 0, s, st, dst_tokens, dst_lens);
    return hipGetLastError();
}

__global__ void turn_over_slots_kernel(StateArgs st, const int* __restrict__ slots, const int* __restrict__ old_reqs,
                                       const int* __restrict__ new_reqs, const int* __restrict__ limits,
                                       const int* __restrict__ all_prompts, int* __restrict__ dst_tokens,
                                       int* __restrict__ dst_lens) {
    const int i = blockIdx.x, tid = threadIdx.x;
    const int b = slots[i], old = old_reqs[i], req = new_reqs[i];
    if (old >= 0) {
        const int n = st.n_gen[b];
        for (int t = tid; t < st.max_new; t += blockDim.x)
            dst_tokens[(size_t)old * st.max_new + t] = t < n ? st.out_tokens[(size_t)b * st.out_stride + t] : st.pad_id;
        if (tid == 0) dst_lens[old] = n;
    }
    __syncthreads();  // n_gen is read above and cleared below
    if (req >= 0)
        for (int p = tid; p < st.prompt_len; p += blockDim.x)
            st.prompt[(size_t)b * st.prompt_stride + p] = all_prompts[(size_t)req * st.prompt_len + p];
    if (tid == 0) {
        st.seq_len[b] = 0;
        st.n_gen[b] = 0;
        st.finished[b] = req < 0;
        st.cur_tok[b] = req >= 0 ? all_prompts[(size_t)req * st.prompt_len] : 0;
        st.limit[b] = req >= 0 ? limits[i] : INT_MAX;
    }
}

hipError_t launch_turn_over_slots(const StateArgs& st, const int* slots, const int* old_reqs, const int* new_reqs,
                                  const int* limits, int n, const int* all_prompts, int* dst_tokens, int* dst_lens,
                                  hipStream_t s) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(turn_over_slots_kernel, dim3(n), dim3(64), 0, s, st, slots, old_reqs, new_reqs, limits,
                       all_prompts, dst_tokens, dst_lens);
    return hipGetLastError();
}

__global__ void assign_pages_kernel(int* __restrict__ page_table, int max_pages, int blk, int first_page, int batch) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < batch) page_table[(size_t)b * max_pages + blk] = first_page + b;
}

hipError_t launch_assign_pages(int* page_table, int max_pages, int blk, int first_page, int batch, hipStream_t s) {
    if (batch < 1 || blk < 0 || blk >= max_pages) return hipErrorInvalidValue;
    hipLaunchKernelGGL(assign_pages_kernel, dim3((batch + 255) / 256), dim3(256), 0, s, page_table, max_pages, blk,
                       first_page, batch);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(int* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_fill_zero(int* p, int n, hipStream_t s) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

__global__ void prepare_timing_kernel(StateArgs st, int max_pos) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = b; i < st.n_items; i += gridDim.x * blockDim.x) st.items[i].x &= ~kItemOff;
    if (b >= st.batch) return;
    st.finished[b] = 0;
    const int p = st.seq_len[b];
    const int pos = p < 0 ? 0 : (p > max_pos ? max_pos : p);
    st.seq_len[b] = pos;
    st.kv_slot[b] = slot_of(st, b, pos);
}

hipError_t launch_prepare_timing(const StateArgs& st, int max_pos, hipStream_t s) {
    hipLaunchKernelGGL(prepare_timing_kernel, dim3((st.batch + 255) / 256), dim3(256), 0, s, st, max_pos);
    return hipGetLastError();
}

}  // namespace aed
