// csrc/kernel_tail.h: where a kernel's tails lie in its arguments, and arguments of every kind out of a tail that lies at any dword.
#include <stdio.h>

#include "kernel_tail.h"

using namespace aed;

FiberIdx::operator unsigned() const { return 0; }
FiberIdx3 threadIdx;
dim3 blockIdx, blockDim, gridDim;
void __syncthreads() {}
uint32_t exchange(uint32_t, int) { return 0; }

struct Args { float f; void* p; int i; const float* q; long long n; int skipped, j; };
// one word beyond a single load, four-byte arguments in front of eight-byte ones
struct Mixed {
    template <typename F> static constexpr void fields(Args& a, F&& f) {
        f(a.f); f(a.p); f(a.i); f(a.q); f(a.n); f(a.j);
        f(a.p); f(a.q); f(a.n); f(a.i); f(a.j);
    }
};
struct Few {
    template <typename F> static constexpr void fields(Args& a, F&& f) { f(a.q); f(a.i); }
};
static_assert(tail_words<Mixed, Args>() == 17 && tail_words<Few, Args>() == 3, "words");
static_assert(TailLoad<Mixed, Args>::kTwo && !TailLoad<Few, Args>::kTwo, "loads");

struct OneTail { const void *a, *b, *c; int m, k, t; ArgTail tail; };
struct TwoTails { const void *a, *b, *c; int m, k; ArgTail t0, t1; };
struct OddTail { const void* a; char b; short c; ArgTail tail; };
static_assert(TailOffset<void(const void*, const void*, const float2*, int, int, int, ArgTail)>::of(0) == offsetof(OneTail, tail), "one");
static_assert(TailOffset<void(const void*, const void*, const void*, int, int, ArgTail, ArgTail)>::of(0) == offsetof(TwoTails, t0), "two");
static_assert(TailOffset<void(const void*, const void*, const void*, int, int, ArgTail, ArgTail)>::of(1) == offsetof(TwoTails, t1), "two");
static_assert(TailOffset<void(const void*, char, short, ArgTail)>::of(0) == offsetof(OddTail, tail), "odd");
static_assert(TailOffset<void(const void*, int)>::of(0) < 0, "none");

template <typename Fields> static int round_trip() {
    alignas(64) char mem[64 + sizeof(ArgTail)];
    int bad = 0;
    for (int at = 0; at < 64; at += 4) {
        Args a = {1.5f, mem, -7, reinterpret_cast<float*>(mem + 8), -(1ll << 40), 3, 11}, b = {};
        const ArgTail t = make_tail<Fields>(a);
        memcpy(mem + at, &t, sizeof t);
        TailLoad<Fields, Args> load((TailPtr)(mem + at));
        load.get(b);
        bad += b.q != a.q || b.i != a.i;
        if (tail_words<Fields, Args>() > 3) bad += b.f != a.f || b.p != a.p || b.n != a.n || b.j != a.j || b.skipped != 0;
    }
    return bad;
}

int main() {
    const int bad = round_trip<Mixed>() + round_trip<Few>();
    printf("%d wrong\n", bad);
    return bad != 0;
}
