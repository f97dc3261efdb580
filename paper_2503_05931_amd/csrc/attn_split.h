// How attention is split over workgroups and wavefronts (host side): which cross-attention sequences are cut into several
// work items, the list of items, and how many wavefronts an item's workgroup has.
#pragma once
#include <limits.h>

#include <algorithm>
#include <vector>

#include "kernels.h"

namespace aed {

// Cross-attention work items.  A sequence of more than `longest` keys is cut into pieces of about `piece` keys.
struct CrossCut { int longest, piece; };
// Batches of more than 4096 are left whole: a CU has 32 workgroups and more then, and with the pieces a prompt pass's list
// (kMaxPrefillPositions times as long) could pass what a launch grid holds in y.
inline CrossCut cross_cut(long long total_keys, int batch, int n_heads, Dtype dt) {
    if (batch > 4096) return CrossCut{INT_MAX, INT_MAX};
    const long long share = total_keys * n_heads / 256 * (dt == kF32 ? 2 : 1);
    CrossCut c;
    c.longest = (int)std::min<long long>(std::max<long long>(192, share * 7 / 8), INT_MAX);
    c.piece = (int)std::min<long long>(std::max<long long>(64, share * 7 / 16 / 32 * 32), INT_MAX);
    return c;
}
inline int cross_pieces(int len, const CrossCut& c) {
    return len <= c.longest ? 1 : std::min(kMaxChunks, (len + c.piece - 1) / c.piece);
}
inline int piece_keys(int len, const CrossCut& c) {
    const int n = cross_pieces(len, c);
    return ((len + n - 1) / n + 15) / 16 * 16;
}
// most keys of an item of a sequence of len keys
inline int item_keys(int len, const CrossCut& c) { return std::min(len, piece_keys(len, c)); }
// the work items of sequence b of len keys, the first at frame first_frame of the packed layout
inline void add_items(std::vector<int4>& items, int b, int len, int first_frame, const CrossCut& c) {
    const int per = piece_keys(len, c), n = (len + per - 1) / per;
    for (int k = 0; k < n; ++k) {
        int4 it;
        it.x = b; it.y = (k * per) | (k << 16); it.z = std::min(per, len - k * per) | (n << 16); it.w = first_frame;
        items.push_back(it);
    }
}
// Cut sequences first, so that their merge is over when the rest is; then longest first.  Stable, so that the list is a
// function of the lengths alone.
inline void order_items(std::vector<int4>& items) {
    std::stable_sort(items.begin(), items.end(), [](const int4& p, const int4& q) {
        const bool pc = p.z >> 16 > 1, qc = q.z >> 16 > 1;
        return pc != qc ? pc : (p.z & 0xFFFF) > (q.z & 0xFFFF);
    });
}

constexpr bool attn_short_items(int most_keys) { return most_keys <= 64; }

// Wavefronts per workgroup, 4 or 8, of a launch of wgs workgroups over caches of kv_bytes an element.  What counts is that
// every workgroup is resident from the start (4096 wavefronts fit the 256 CUs, of float32 rows 2048) and that a wavefront has
// a block or two to itself: with 8 wavefronts where 8 do not fit, a second round of workgroups starts when the first is over
// (self-attention, 24 layers, batch 128, 33 positions: 44.4 ms with 8, 42.9 with 4; batch 64 125.0 and 125.4 for 131), and
// wavefronts without a block still cost the merge (one utterance, cross- and self-attention on 16 and on 4: 92.6 and 90.1 ms).
// Items that are long on average (kLongItem) keep memory busy in two rounds as well, and 8 wavefronts are through with the last
// ones sooner (24 layers, batch 128 of 12 to 500 frames, half of whose sequences are through on average: 357 and 350 ms).
// 16 are nowhere better than 8 (bfloat16, 8 heads of 128, us a launch on 16 / 8 / 4: cross-attention of 350 keys, batch 16 8.8 /
// 8.1 / 8.1, batch 32 11.4 / 10.6 / 10.3; 500 keys 11.3 / 9.7 / 10.1 and 15.1 / 13.3 / 13.4; self-attention over 440 positions,
// batch 16 8.4 / 7.9 / 7.8, batch 32 11.6 / 11.1 / 11.0; 4 heads of 64, 500 keys, batch 64 9.1 / 7.7 / 8.0): the keys of 8 are as
// many as a CU has under way, and the merge of 16 takes longer.
// Items of at most 64 keys are 4 blocks.  (Taken for as long as a sequence that is just not cut, they had 8: one utterance of
// 200 / 350 / 500 keys 5.18 / 5.27 / 5.40 us, 5.12 / 5.19 / 5.32 on 4; 8-bit caches, batch 16 of 200 keys 7.7 and 6.8.)
inline int attn_wavefronts(size_t wgs, int kv_bytes, int most_keys, bool long_items) {
    const size_t resident = kv_bytes <= 2 ? 4096 : 2048;
    return wgs * 8 > (long_items ? 2 * resident : resident) || attn_short_items(most_keys) ? 4 : 8;
}

}  // namespace aed
