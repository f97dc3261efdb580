// Kernel arguments on two ways.  What a workgroup needs before its first request to memory is passed as leading scalar
// arguments: they arrive in registers with the wavefront (-amdgpu-kernarg-preload-count in build.py).  Anything else is
// fetched from memory by the kernel, a trip in front of everything that waits for it; it is packed into a tail, which one or
// two wide scalar loads bring: asked for when the kernel starts, used when the first requests are out.  (Of a struct read field
// by field the compiler asks for each field where it is used, one trip after the other, or waits for all in front of the first
// request.)  A graph of 168 launches of 256 workgroups that stream 32 KB each, in us a launch: a struct of arguments 3.15, leading
// scalars preloaded 2.77; 4 KB each 1.86 and 2.00, because the launch itself takes 0.1 us longer then.  The streaming products
// and attention, whole decodes before -> with it: 24 layers, batch 1, 3 x 40 tokens 85.0 -> 77.9 ms, batch 64, 128 tokens 123.4 ->
// 117.0, batch 16 with logits 22.4 -> 21.5; 4 layers, batch 256, 128 tokens 41.2 -> 40.1.
#pragma once

#include <string.h>

#include <type_traits>

#include "common.h"

namespace aed {

constexpr int kTailWords = 32;
struct alignas(8) ArgTail { unsigned w[kTailWords]; };
typedef unsigned u32x16 __attribute__((ext_vector_type(16)));
typedef u32x16 u32x16_packed __attribute__((aligned(4)));  // a tail begins where the leading arguments end; scalar loads take any dword
typedef const __attribute__((address_space(4))) u32x16_packed* TailPtr;
// Where the tails of a kernel lie in its arguments: its function type's arguments one after the other, each at its own alignment
template <typename Kernel> struct TailOffset;
template <typename... A> struct TailOffset<void(A...)> {
    static constexpr int of(int which) {
        const int size[] = {(int)sizeof(A)...}, align[] = {(int)alignof(A)...};
        const bool tail[] = {std::is_same<A, ArgTail>::value...};
        int at = 0;
        for (int i = 0; i < (int)sizeof...(A); ++i) {
            at = (at + align[i] - 1) / align[i] * align[i];
            if (tail[i] && which-- == 0) return at;
            at += size[i];
        }
        return -1;
    }
};
template <typename Kernel, int Which = 0> __device__ __forceinline__ TailPtr tail_of() {
    constexpr int offset = TailOffset<Kernel>::of(Which);
    static_assert(offset >= 0, "the kernel has no such tail");
#if defined(__HIP_DEVICE_COMPILE__)
    return (TailPtr)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + offset);
#else
    return nullptr;
#endif
}
// nothing uses v, a value in scalar registers, before this
template <typename V> __device__ __forceinline__ void settle(V& v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v));
#endif
}

// pointers are to memory: without saying so their uses become flat accesses, which every wait for LDS waits for
template <typename V> __device__ __forceinline__ void set_field(V*& p, unsigned long long bits) {
    p = (V*)(__attribute__((address_space(1))) V*)bits;
}
__device__ __forceinline__ void set_field(long long& v, unsigned long long bits) { v = (long long)bits; }
__device__ __forceinline__ void set_field(int& v, unsigned bits) { v = (int)bits; }
__device__ __forceinline__ void set_field(float& v, unsigned bits) { v = __builtin_bit_cast(float, bits); }

// Fields: a type with a constexpr fields(Args&, f), which calls f for every argument in the tail
struct TailCounter {
    int words = 0;
    template <typename V> constexpr void operator()(V&) {
        static_assert(sizeof(V) == 8 || sizeof(V) == 4, "pointers, long long, int, float");
        words += sizeof(V) / 4;
    }
};
template <typename Fields, typename Args> constexpr int tail_words() {
    Args a{};
    TailCounter c;
    Fields::fields(a, c);
    return c.words;
}
template <typename Fields, typename Args> static ArgTail make_tail(Args a) {
    static_assert(tail_words<Fields, Args>() <= kTailWords, "a tail is at most two scalar loads");
    ArgTail t = {};
    size_t at = 0;
    Fields::fields(a, [&](auto& v) {
        memcpy(reinterpret_cast<char*>(t.w) + at, &v, sizeof v);
        at += sizeof v;
    });
    return t;
}

template <typename Fields, typename Args> struct TailLoad {
    static constexpr bool kTwo = tail_words<Fields, Args>() > 16;
    u32x16 lo, hi;
    __device__ __forceinline__ explicit TailLoad(TailPtr p) {
        lo = p[0];
        if constexpr (kTwo) hi = p[1];
    }
    // the arguments; nothing uses them before this
    __device__ __forceinline__ void get(Args& a) {
        settle(lo);
        if constexpr (kTwo) settle(hi);
        int at = 0;
        auto word = [&](int i) { return i < 16 ? lo[i & 15] : hi[i & 15]; };
        Fields::fields(a, [&](auto& v) {
            if constexpr (sizeof v == 8) {
                set_field(v, (unsigned long long)word(at) | (unsigned long long)word(at + 1) << 32);
                at += 2;
            } else {
                set_field(v, word(at));
                at += 1;
            }
        });
    }
};

}  // namespace aed
