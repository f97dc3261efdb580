// One workgroup of a step's last kernel (csrc/step_kernels.hip, unchanged) on the
// CPU, with its wavefronts run one after the other in a given order, each until it
// ends or waits.  The hardware promises no order between two barriers, so state, work
// list and the embedded row must come out the same in all of them.  Inside a wavefront the lanes
// run from the last to the first: lane 0, which stores, comes after the others' loads,
// as in lockstep.
#include <math.h>
#include <stdio.h>
#include <string.h>
#include <ucontext.h>

#include <vector>

#include "step_kernels.hip"

namespace {
constexpr int kThreads = 256;
enum What { READY, BARRIER, EXCHANGE, ENDED };
struct Fiber { ucontext_t ctx; What what; uint32_t sent; std::vector<char> stack; };
Fiber fibers[kThreads];
ucontext_t scheduler;
int current;
void (*body)();

void run_body() {
    body();
    fibers[current].what = ENDED;
}
void wait_at(What w) {
    fibers[current].what = w;
    swapcontext(&fibers[current].ctx, &scheduler);
}
void run_workgroup(void (*f)(), const int* wave_order) {
    body = f;
    for (Fiber& x : fibers) {
        x.what = READY;
        x.stack.resize(64 << 10);
        getcontext(&x.ctx);
        x.ctx.uc_stack.ss_sp = x.stack.data();
        x.ctx.uc_stack.ss_size = x.stack.size();
        x.ctx.uc_link = &scheduler;
        makecontext(&x.ctx, run_body, 0);
    }
    auto all = [](int t0, int n, What w) {  // of the threads that still run; false if there are none
        int live = 0;
        for (int t = t0; t < t0 + n; ++t) {
            if (fibers[t].what == ENDED) continue;
            if (fibers[t].what != w) return false;
            ++live;
        }
        return live > 0;
    };
    for (;;) {
        for (int i = 0; i < 4; ++i) {
            const int t0 = 64 * wave_order[i];
            for (;;) {  // this wavefront as far as it goes
                for (int t = t0 + 63; t >= t0; --t)
                    if (fibers[t].what == READY) {
                        current = t;
                        swapcontext(&scheduler, &fibers[t].ctx);
                    }
                if (!all(t0, 64, EXCHANGE)) break;
                for (int t = t0; t < t0 + 64; ++t)
                    if (fibers[t].what == EXCHANGE) fibers[t].what = READY;
            }
        }
        if (!all(0, kThreads, BARRIER)) break;
        for (Fiber& x : fibers)
            if (x.what == BARRIER) x.what = READY;
    }
    for (const Fiber& x : fibers)
        if (x.what != ENDED) { printf("a thread never ended\n"); __builtin_trap(); }
}

// the kernels' operands: four sequences, the second is the one that is run
constexpr int kSeqs = 4, kSeq = 1, kVocab = 512, kMaxNew = 8, kPrompt = 14, kItems = 150, kPos = 18, kDim = 320, kPages = 2;
template <typename T> struct World {
    int seq_len[kSeqs], n_gen[kSeqs], finished[kSeqs], cur_tok[kSeqs], limit[kSeqs], n_finished;
    int prompt[kSeqs * kPrompt], out[kSeqs * 16], pages[kSeqs * kPages], kv_slot[kSeqs], step_out[kSeqs];
    int4 items[kItems];
    alignas(16) float logits[kSeqs * kVocab], x[16 * kDim];
    alignas(16) T tok[kVocab * kDim], pos[kPos * kDim], shadow[16 * kDim];
    float2 stats[kSeqs * kDim / 16];
    float mu_hat[kSeqs];
};
template <typename T> World<T> world;
aed::StateArgs args;
aed::EmbedArgs emb;
template <typename T> void greedy_end() { aed::sample_embed_kernel<T>(world<T>.logits, args, emb); }
template <typename T> void step_end() { aed::sample_kernel(world<T>.logits, args, world<T>.step_out); }

template <typename T> void fill(int pos, int n, int limit, int max_new, int best, bool finished, bool shadow, bool rms) {
    World<T>& w = world<T>;
    memset(&w, 0, sizeof w);
    for (int i = 0; i < kSeqs * kVocab; ++i) w.logits[i] = (float)((i * 37) % 101);
    w.logits[kSeq * kVocab + best] = 1000.f;
    for (int i = 0; i < kVocab * kDim; ++i) w.tok[i] = (T)(float)((i * 29 % 251) / 32.f);  // bfloat16 has these exactly
    for (int i = 0; i < kPos * kDim; ++i) w.pos[i] = (T)(float)((i * 53 % 127) / 16.f);
    for (int b = 0; b < kSeqs; ++b) {
        w.seq_len[b] = pos;
        w.n_gen[b] = n;
        w.limit[b] = limit;
        w.cur_tok[b] = 40 + b;
        w.kv_slot[b] = -7;
        for (int p = 0; p < kPrompt; ++p) w.prompt[b * kPrompt + p] = 16 * b + p;
        for (int p = 0; p < kPages; ++p) w.pages[b * kPages + p] = 10 * b + 3 * p + 1;
    }
    w.finished[kSeq] = finished;
    for (int i = 0; i < kItems; ++i) w.items[i].x = i % 3;  // the list takes more than one wavefront
    args = aed::StateArgs{};
    args.seq_len = w.seq_len; args.n_gen = w.n_gen; args.finished = w.finished;
    args.cur_tok = w.cur_tok; args.limit = w.limit; args.n_finished = &w.n_finished;
    args.prompt = w.prompt; args.out_tokens = w.out; args.page_table = w.pages; args.max_pages = kPages; args.kv_slot = w.kv_slot;
    args.prompt_len = kPrompt; args.prompt_stride = kPrompt; args.out_stride = 16; args.max_new = max_new;
    args.eos_id = 2; args.pad_id = 0; args.batch = kSeqs; args.vocab = kVocab;
    args.items = w.items; args.n_items = kItems;
    emb = aed::EmbedArgs{};
    emb.x = w.x; emb.tok_emb = w.tok; emb.pos_emb = w.pos; emb.d = kDim; emb.max_positions = kPos; emb.emb_scale = 3.f;
    emb.sh.stats = w.stats;
    if (shadow) { emb.sh.shadow = w.shadow; emb.sh.mu_hat = w.mu_hat; emb.sh.rms = rms; }
}

// the row that sequence kSeq feeds next: token tok at position pos, cached in slot
template <typename T> bool embedded(int tok, int pos, int slot) {
    const World<T>& w = world<T>;
    const int at = std::min(pos, kPos - 1);
    double o[kDim], mean = 0;
    for (int k = 0; k < kDim; ++k) {
        o[k] = 3. * (float)w.tok[tok * kDim + k] + (float)w.pos[at * kDim + k];
        mean += o[k] / kDim;
    }
    bool ok = w.kv_slot[kSeq] == slot && w.kv_slot[0] == -7;
    // float32 sums of 320 values of at most 32: 320 * 2^-24 * 32 relative to the largest
    auto near = [](double a, double b) { return fabs(a - b) <= 7e-4; };
    for (int k = 0; k < kDim; ++k) ok = ok && w.x[aed::frag_elem_off<4>(kSeq, k, kDim) / 4] == (float)o[k];
    for (int t = 0; t < kDim / 16; ++t) {
        double m = 0, q = 0;
        for (int k = 0; k < 16; ++k) m += o[16 * t + k] / 16;
        for (int k = 0; k < 16; ++k) q += (o[16 * t + k] - m) * (o[16 * t + k] - m);
        ok = ok && near(w.stats[kSeq * kDim / 16 + t].x, m) && fabs(w.stats[kSeq * kDim / 16 + t].y - q) <= 1e-5 * q + 1e-3;
    }
    if (!emb.sh.shadow) return ok;
    const double shift = emb.sh.rms ? 0 : mean;
    ok = ok && near(w.mu_hat[kSeq], shift);
    for (int k = 0; k < kDim; ++k) {
        const double v = (float)w.shadow[aed::frag_elem_off<sizeof(T)>(kSeq, k, kDim) / sizeof(T)];
        ok = ok && fabs(v - (o[k] - shift)) <= fabs(o[k] - shift) / 256 + 7e-4;  // rounded to 8 bits
    }
    return ok;
}
}  // namespace

FiberIdx::operator unsigned() const { return (unsigned)current; }
FiberIdx3 threadIdx;
dim3 blockIdx(kSeq), blockDim(kThreads), gridDim(kSeqs);
void __syncthreads() { wait_at(BARRIER); }
uint32_t exchange(uint32_t v, int lane_xor) {
    // twice: the value is read when all lanes have sent theirs, and sent anew only when all have read
    fibers[current].sent = v;
    wait_at(EXCHANGE);
    const uint32_t got = fibers[current ^ lane_xor].sent;
    wait_at(EXCHANGE);
    return got;
}

const int orders[][4] = {{0, 1, 2, 3}, {3, 2, 1, 0}, {1, 0, 3, 2}, {2, 3, 0, 1}};

// pos: position just decoded; max_new / limit: how many tokens the sequence may emit
template <typename T> int run(bool shadow, bool rms) {
    const World<T>& w = world<T>;
    int bad = 0;
    for (int pos = kPrompt - 3; pos < kPos; ++pos)
        for (int max_new = 1; max_new <= kMaxNew; max_new += 7)
            for (int limit = 1; limit <= 9; limit += 4)
                for (int kind = 0; kind < 4; ++kind)  // goes on, emits the end, had ended before, a step's end
                    for (const int* order : orders) {
                        const bool finished = kind == 2, step = kind == 3, feeding = !step && pos + 1 < kPrompt;
                        const int n = feeding ? 0 : std::max(0, pos + 1 - kPrompt);
                        if (!feeding && !finished && !step && (n >= max_new || n >= limit)) continue;  // such a sequence has ended before
                        const int best = kind == 1 ? 2 : 300;
                        fill<T>(pos, n, limit, max_new, best, finished, shadow, rms);
                        run_workgroup(step ? step_end<T> : greedy_end<T>, order);

                        const bool moves = !finished, emits = moves && !feeding;
                        const int tok = !step && n + 1 >= limit ? 2 : best;
                        const bool ends = emits && !step && (tok == 2 || n + 1 >= max_new);
                        const int fed = finished ? 40 + kSeq : feeding ? 16 * kSeq + pos + 1 : tok, next = pos + moves;
                        bool ok = w.seq_len[kSeq] == next && w.seq_len[0] == pos && w.cur_tok[kSeq] == fed;
                        ok = ok && w.n_gen[kSeq] == n + (emits && !step) && w.finished[kSeq] == (finished || ends) && w.n_finished == ends;
                        ok = ok && (!emits || step || w.out[16 * kSeq + n] == tok) && w.step_out[kSeq] == (step ? tok : 0);
                        for (int i = 0; i < kItems; ++i) ok = ok && (w.items[i].x < 0) == (ends && i % 3 == kSeq);
                        const int at = std::min(next, kPos - 1);
                        if (!step) ok = ok && embedded<T>(fed, next, finished || ends ? -1 : w.pages[kSeq * kPages + at / 16] * 16 + at % 16);
                        if (!ok) {
                            printf("position %d of a prompt of %d, max_new %d, limit %d, kind %d, wavefronts %d %d %d %d: "
                                   "finished %d, token %d, slot %d, items off:", pos, kPrompt, max_new, limit, kind, order[0], order[1],
                                   order[2], order[3], w.finished[kSeq], w.cur_tok[kSeq], w.kv_slot[kSeq]);
                            for (int i = 0; i < kItems; ++i)
                                if (w.items[i].x < 0) printf(" %d", i);
                            printf("\n");
                            ++bad;
                        }
                    }
    return bad;
}

int main() {
    const int bad = run<float>(false, false) + run<aed::bf16_t>(true, false) + run<aed::bf16_t>(true, true);
    printf("%d wrong\n", bad);
    return bad != 0;
}
