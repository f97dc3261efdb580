// The rules of csrc/attn_split.h over many batches: every key in one item, lists that fit what holds them, and the choices
// themselves where they change over.
#include <stdio.h>

#include "attn_split.h"

using namespace aed;

FiberIdx::operator unsigned() const { return 0; }
FiberIdx3 threadIdx;
dim3 blockIdx, blockDim, gridDim;
void __syncthreads() {}
uint32_t exchange(uint32_t, int) { return 0; }

static int bad = 0;
static void expect(bool ok, const char* what, long long a, long long b, long long c) {
    if (!ok && bad++ < 20) printf("%s: %lld, %lld, %lld\n", what, a, b, c);
}
static unsigned seed = 1;
static unsigned rnd(unsigned n) { seed = seed * 1664525u + 1013904223u; return (seed >> 8) % n; }

static std::vector<int4> list_of(const std::vector<int>& lens, const CrossCut& cut) {
    std::vector<int4> items;
    int at = 0;
    for (size_t b = 0; b < lens.size(); ++b) {
        add_items(items, (int)b, lens[b], at, cut);
        at += lens[b];
    }
    order_items(items);
    return items;
}
static long long sum(const std::vector<int>& v) {
    long long s = 0;
    for (int x : v) s += x;
    return s;
}

static CrossCut cut_of(const std::vector<int>& lens, int heads, int kv) {
    return cross_cut(sum(lens), *std::max_element(lens.begin(), lens.end()), (int)lens.size(), heads, kv);
}
static void check_list(const std::vector<int>& lens, int heads, int kv) {
    const int B = (int)lens.size();
    const long long total = sum(lens);
    const CrossCut cut = cut_of(lens, heads, kv);
    const std::vector<int4> items = list_of(lens, cut);
    // the list has room for every 64 frames and every sequence; a prompt pass repeats it for 8 positions in one grid's y
    expect((long long)items.size() <= total / 64 + B, "more items than the list holds", items.size(), total, B);
    expect(B > 4096 ? (int)items.size() == B : items.size() * 8 <= 65535, "more items than a prompt pass's grid", items.size(), B, heads);
    std::vector<int> covered(B, 0), pieces(B, 0);
    std::vector<int> first(B, 0);
    int most = 0;
    for (int b = 1; b < B; ++b) first[b] = first[b - 1] + lens[b - 1];
    for (size_t i = 0; i < items.size(); ++i) {
        const int b = items[i].x, start = items[i].y & 0xFFFF, idx = items[i].y >> 16, n = items[i].z & 0xFFFF, of = items[i].z >> 16;
        expect(b >= 0 && b < B && n >= 1 && of >= 1 && of <= kMaxChunks && idx >= 0 && idx < of, "item fields", i, idx, of);
        expect(items[i].w == first[b], "first frame", i, items[i].w, first[b]);
        expect(of == 1 || start % 16 == 0, "a piece starts inside a block", i, start, n);
        expect(start + n <= lens[b], "past the sequence's end", b, start + n, lens[b]);
        expect(start == idx * piece_keys(lens[b], cut), "start", b, start, idx);
        covered[b] += n;
        pieces[b] += 1;
        most = std::max(most, n);
        if (i) {
            const bool cut_before = items[i - 1].z >> 16 > 1, cut_now = of > 1;
            expect(cut_before >= cut_now && (cut_before != cut_now || (items[i - 1].z & 0xFFFF) >= n), "order", i, cut_before, cut_now);
        }
    }
    int said = 0;
    for (int len : lens) said = std::max(said, item_keys(len, cut));
    expect(said == most, "most keys of an item", said, most, B);
    std::vector<int> of(B, 0);
    for (const int4& it : items) of[it.x] = it.z >> 16;
    for (int b = 0; b < B; ++b) expect(covered[b] == lens[b] && of[b] == pieces[b], "keys and pieces", b, covered[b], of[b]);
}

int main() {
    // lists of every kind of batch
    for (int heads : {2, 4, 8, 16})
        for (int kv : {1, 2, 4})
            for (int B : {1, 2, 3, 7, 8, 12, 13, 16, 24, 31, 32, 33, 36, 63, 64, 65, 100, 128, 255, 256, 700, 1024, 4096, 4097, 8191})
                for (int kind = 0; kind < 6; ++kind) {
                    std::vector<int> lens(B);
                    for (int b = 0; b < B; ++b)
                        lens[b] = kind == 0 ? 500 : kind == 1 ? 1 + (int)rnd(500) : kind == 2 ? 1 + (int)rnd(64) : kind == 3 ? (b == B / 2 ? 65535 : 1)
                                  : kind == 4 ? 300 + (int)rnd(201) : (rnd(6) ? 1 + (int)rnd(80) : 193 + (int)rnd(3000));
                    check_list(lens, heads, kv);
                }
    for (int len : {1, 63, 64, 65, 191, 192, 193, 256, 257, 511, 512, 513, 2047, 2048, 2049, 65535}) check_list({len}, 4, 2);
    // the longest sequence that is taken, whole: its count fills the item's field
    {
        std::vector<int> lens(4097, 1);
        lens[7] = 65535;
        const std::vector<int4> items = list_of(lens, cut_of(lens, 2, 2));
        expect(items[0].x == 7 && (items[0].y & 0xFFFF) == 0 && items[0].z == (65535 | (1 << 16)), "65535 keys whole", items[0].x, items[0].y, items[0].z);
    }
    // single utterances come out in pieces of at most 64 keys
    for (int len : {193, 300, 400, 500, 512}) expect(item_keys(len, cut_of({len}, 8, 2)) <= 64, "one utterance's pieces", len, 0, 0);
    // balanced batches of one workgroup a CU stay whole, but for few sequences and float32; one long sequence among them is cut
    for (int heads : {4, 8, 16})
        for (int kv : {1, 2, 4})
            for (int B = 1; B <= 300 / heads; ++B)
                for (int len : {193, 350, 500}) {
                    std::vector<int> lens(B, len);
                    lens[B / 2] = len * 5 / 4;
                    const bool whole = kv <= 2 && B * heads > 48 * kv && B * heads <= 256;
                    expect(!whole || (int)list_of(lens, cut_of(lens, heads, kv)).size() == B, "a balanced batch is cut", B, heads, kv);
                    lens[B / 2] = len * 6;
                    expect(B < 4 || B * heads > 256 || (int)list_of(lens, cut_of(lens, heads, kv)).size() > B, "the long one is not", B, heads, kv);
                }
    // float32: one long sequence in ten of a large batch is cut
    for (int B : {65, 80, 96, 128}) {
        std::vector<int> lens(B, 80);
        for (int b = 0; b < B; b += 10) lens[b] = 500;
        expect((int)list_of(lens, cut_of(lens, 8, 4)).size() > B, "long float32 sequences are not cut", B, 0, 0);
    }
    // wavefronts: 8 while 8 are resident (twice that of long items), 4 beyond and for short items
    struct { long wgs; long long pairs; int kv, keys, lng, even, want; } nw[] = {
        {8, 8, 2, 500, 0, 0, 8}, {8, 8, 2, 64, 0, 1, 4}, {8, 8, 2, 65, 0, 1, 8}, {256, 256, 2, 500, 1, 1, 8}, {512, 512, 2, 100, 0, 0, 8},
        {513, 512, 2, 100, 0, 0, 4}, {1024, 1024, 2, 400, 1, 0, 8}, {1025, 1024, 2, 400, 1, 0, 4}, {512, 512, 1, 100, 0, 0, 8},
        {513, 512, 1, 100, 0, 0, 4}, {512, 0, 2, 400, 0, 0, 8}, {513, 0, 2, 400, 0, 0, 4},
        // float32: two rounds of 8 of uneven lengths, whatever the pieces make of them, and of long items; one in self-attention
        {256, 256, 4, 500, 0, 1, 8}, {300, 200, 4, 100, 0, 0, 4}, {300, 257, 4, 100, 0, 0, 8}, {300, 257, 4, 100, 0, 1, 4}, {700, 512, 4, 100, 0, 0, 8},
        {700, 512, 4, 64, 0, 0, 4}, {700, 513, 4, 100, 0, 0, 4}, {512, 600, 4, 400, 1, 0, 8}, {513, 600, 4, 400, 1, 0, 4}, {256, 0, 4, 400, 0, 0, 8},
        {257, 0, 4, 400, 0, 0, 4}};
    for (const auto& c : nw) {
        const int got = attn_wavefronts(c.wgs, c.pairs, c.kv, c.keys, c.lng, c.even);
        expect(got == c.want, "wavefronts", c.wgs, got, c.want);
    }
    // the frames instead of keys and values: 288 sequences and more of more than about 350 to 220 frames, the longest no longer than a
    // CU's share of all; a decoder that has no room for 140 * 288 + 60 000 frames has no such batch
    struct { long long total; int longest, batch; bool want; } frames[] = {
        {140 * 288 + 60000, 390, 288, true}, {140 * 288 + 59999, 390, 288, false}, {1 << 20, 500, 287, false}, {140 * 288 + 60000, 392, 288, false},
        {512 * 500, 500, 512, true}, {1024 * 500, 500, 1024, true}, {1024 * 500, 2000, 1024, true}, {1024 * 500, 2001, 1024, false},
        {1024 * 150, 200, 1024, false}, {1024 * 250, 300, 1024, true}, {65535ll * 65535, 65535, 65535, true}};
    for (const auto& c : frames) expect(frames_attention(c.total, c.longest, c.batch) == c.want, "frames", c.total, c.longest, c.batch);
    for (int B = kFramesMinBatch; B < 5000; ++B) expect(frames_min_keys(B) >= frames_min_keys(kFramesMinBatch), "least frames", B, 0, 0);
    printf("%d wrong\n", bad);
    return bad != 0;
}
