// One workgroup of the greedy sampler (csrc/step_kernels.hip, unchanged) on the
// CPU, with its wavefronts run one after the other in a given order, each until it
// ends or waits.  The hardware promises no order between two barriers, so state and
// work list must come out the same in all of them.  Inside a wavefront the lanes
// run from the last to the first: lane 0, which stores, comes after the others' loads,
// as in lockstep.
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

// the sampler's operands: four sequences, the second is the one that is run
constexpr int kSeqs = 4, kSeq = 1, kVocab = 512, kMaxNew = 8, kPrompt = 5, kItems = 150;
struct World {
    int seq_len[kSeqs], n_gen[kSeqs], finished[kSeqs], cur_tok[kSeqs], limit[kSeqs], n_finished;
    int prompt[kSeqs * kPrompt], out[kSeqs * 16];
    int4 items[kItems];
    alignas(16) float logits[kSeqs * kVocab];
} world;
aed::StateArgs args;
void sample() { aed::sample_kernel(world.logits, args, 1, nullptr); }
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

int main() {
    const int orders[][4] = {{0, 1, 2, 3}, {3, 2, 1, 0}, {1, 0, 3, 2}, {2, 3, 0, 1}};
    int bad = 0;
    // pos: position just decoded; max_new / limit: how many tokens the sequence may emit
    for (int pos = 0; pos < kPrompt + 3; ++pos)
        for (int max_new = 1; max_new <= kMaxNew; max_new += 7)
            for (int limit = 1; limit <= 9; limit += 4)
                for (int emits_eos = 0; emits_eos < 2; ++emits_eos)
                    for (const int* order : orders) {
                        const bool feeding = pos + 1 < kPrompt;
                        const int n = feeding ? 0 : pos + 1 - kPrompt;
                        if (!feeding && (n >= max_new || n >= limit)) continue;  // such a sequence has ended before
                        memset(&world, 0, sizeof world);
                        for (int i = 0; i < kSeqs * kVocab; ++i) world.logits[i] = (float)((i * 37) % 101);
                        const int best = emits_eos ? 2 : 300;
                        world.logits[kSeq * kVocab + best] = 1000.f;
                        for (int b = 0; b < kSeqs; ++b) {
                            world.seq_len[b] = pos;
                            world.n_gen[b] = n;
                            world.limit[b] = limit;
                            for (int p = 0; p < kPrompt; ++p) world.prompt[b * kPrompt + p] = 10 * b + p;
                        }
                        for (int i = 0; i < kItems; ++i) world.items[i].x = i % 3;  // the list takes more than one wavefront
                        args = aed::StateArgs{};
                        args.seq_len = world.seq_len; args.n_gen = world.n_gen; args.finished = world.finished;
                        args.cur_tok = world.cur_tok; args.limit = world.limit; args.n_finished = &world.n_finished;
                        args.prompt = world.prompt; args.out_tokens = world.out;
                        args.prompt_len = kPrompt; args.prompt_stride = kPrompt; args.out_stride = 16; args.max_new = max_new;
                        args.eos_id = 2; args.pad_id = 0; args.batch = kSeqs; args.vocab = kVocab;
                        args.items = world.items; args.n_items = kItems;
                        run_workgroup(sample, order);

                        const int tok = n + 1 >= limit ? 2 : best;
                        const bool ends = !feeding && (tok == 2 || n + 1 >= max_new);
                        bool ok = world.seq_len[kSeq] == pos + 1 && world.seq_len[0] == pos;
                        ok = ok && world.cur_tok[kSeq] == (feeding ? 10 * kSeq + pos + 1 : tok);
                        ok = ok && world.n_gen[kSeq] == (feeding ? 0 : n + 1) && world.finished[kSeq] == ends && world.n_finished == ends;
                        ok = ok && (feeding || world.out[16 * kSeq + n] == tok);
                        for (int i = 0; i < kItems; ++i) ok = ok && (world.items[i].x < 0) == (ends && i % 3 == kSeq);
                        if (!ok) {
                            printf("position %d of a prompt of %d, max_new %d, limit %d, wavefronts %d %d %d %d: "
                                   "finished %d, items off:", pos, kPrompt, max_new, limit, order[0], order[1], order[2], order[3],
                                   world.finished[kSeq]);
                            for (int i = 0; i < kItems; ++i)
                                if (world.items[i].x < 0) printf(" %d", i);
                            printf("\n");
                            ++bad;
                        }
                    }
    printf("%d wrong\n", bad);
    return bad != 0;
}
